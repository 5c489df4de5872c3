// Pieces shared by the three forms of the attention kernel (attend.hip: 256 query rows and eight wavefronts per
// workgroup, or 128 rows and four; attend_split.hip: 128 query rows per workgroup with the keys of every tile split over
// two groups of wavefronts): launch arguments, the tile generator that walks plain causal tiles or a block list,
// the half-tile products on v_mfma_f32_32x32x16_bf16 and the online-softmax steps.
#pragma once

#include "tsa_internal.h"

#include <climits>

namespace tsa {

namespace attend_detail {

constexpr int BM = 256;        // query rows per workgroup
constexpr int BN = kKeyTile;   // keys per tile
#ifndef TSA_PF
#define TSA_PF 3
#define TSA_RING 4
#endif
#ifndef TSA_QS
#define TSA_QS 1
#endif


constexpr int kQS = TSA_QS;    // query sub-tiles per wavefront (see attend_kernel)
constexpr int kMaxLists = BM / BN;   // row blocks of a query tile at the smallest block size (64): 4
constexpr float kNegBig = -1.0e30f;
constexpr float kLazy = 8.0f;  // log2 units the running max may lag behind

struct AttendArgs {
  const __bf16* Q;
  const __bf16* K;
  const __bf16* Vt;            // tiled V^T: [B * kvh][nk_tiles][d][64]
  __bf16* O;
  float* lse;
  const int32_t* block_list;
  long long bl_head_stride;    // elements between the block lists of consecutive (b, h); 0 = one shared list
  int max_blocks;
  int block;                   // block size of the list: 64, 128 or 256 tokens
  int BH, Hq, kvh, Lc, nq_tiles, nk_tiles;
  int split_log2, vheads_per_xcd;   // workgroup -> (head, query tile) map, see map_workgroups()
  FastDiv by_vheads, by_Hq;    // ... its divisions
  FastDiv by_g, by_g_kv;       // query heads per head of V^ (and index set), per head of K
  const int32_t* k_dev;        // fused form: compacted rows per batch entry, decided on the device (NULL: Lc)
  Strides qs, ks, os;          // fused form: layouts of the original Q, K and of the full-length output (elements)
  float c;                     // scale * log2(e)
  // Fused form (gather in the loads, scatter in the epilogue): Q and K are the ORIGINAL tensors of
  // L tokens (K with Hkv heads), compacted row r of selection row `sel` is token idx[sel][r];
  // Vt holds the tiles of the gathered V.  Of (may be NULL) is the full-length output
  // [B,Hq,L,d]: rows of selected tokens are written by the epilogue, all other rows are
  // zero-filled by the workgroup that owns their token range (inv[sel][t] < 0).  O (the compacted
  // output) may be NULL in this form.
  // X (may be NULL) is the residual stream [B,L,Hq*d]: the epilogue adds output row r, as rounded
  // to bf16, into X[b, idx[r], h*d .. (h+1)*d) (fp32 add, one rounding); every (token, head) slice
  // has exactly one writer.
  const int32_t* idx;
  const int32_t* inv;
  __bf16* Of;
  __bf16* X;
  int L, Hkv;
};

// Workgroup -> (head, query tile).  Consecutive workgroup ids go to different XCDs, so id % 8 picks the XCD.
// A head's query tiles stay on one XCD (they stream the same K / V through its L2), consecutive heads (the
// heads of a KV group) share an XCD, and the longest (last) query tiles are scheduled first.  When the number
// of heads is no multiple of 8, whole heads per XCD would leave some XCDs with one head more than others (28
// heads: four against three, a launch 14 % longer than its work); every head is then cut into
// 1 << split_log2 parts (query tiles qt with (nq - 1 - qt) % parts == part; 2, 4 or 8 of them), so that all the parts
// divide evenly: XCD x takes parts [x * vheads_per_xcd, (x + 1) * vheads_per_xcd), i.e. whole heads and at
// most two partial ones.
inline void map_workgroups(AttendArgs& a) {
  int g = 8, log2 = 0;
  while (a.BH % g) { g >>= 1; ++log2; }           // gcd(BH, 8)
  a.split_log2 = log2;
  a.vheads_per_xcd = a.BH / g;
  const uint64_t heads = (uint64_t)a.BH;
  a.by_vheads = FastDiv(a.vheads_per_xcd, (uint64_t)a.vheads_per_xcd * (a.nq_tiles + 1));
  a.by_Hq = FastDiv(a.Hq, heads);
  a.by_g = FastDiv(a.Hq / a.kvh, a.Hq);
  a.by_g_kv = FastDiv(a.Hq / a.Hkv, a.Hq);
}
inline unsigned grid_for(const AttendArgs& a) {
  return 8u * (unsigned)a.vheads_per_xcd * (unsigned)((a.nq_tiles + (1 << a.split_log2) - 1) >> a.split_log2);
}

// The map on the device: head b, h and the number of the query tile counted from the last one.
__device__ __forceinline__ void workgroup_of(const AttendArgs& a, unsigned id, int& b, int& h, int& from_last) {
  const unsigned xcd = id & 7u, slot = id >> 3;
  const unsigned rank = a.by_vheads.div(slot), vhead = xcd * a.vheads_per_xcd + (slot - rank * a.vheads_per_xcd);
  const unsigned hp = vhead >> a.split_log2, part = vhead & ((1u << a.split_log2) - 1u);
  const unsigned b_ = a.by_Hq.div(hp);
  b = (int)b_;
  h = (int)(hp - b_ * a.Hq);
  from_last = (int)((rank << a.split_log2) + part);
}
// First token of query tile t's share of the zero rows, of nq tiles (see attend.hip): one function of the tile for both
// neighbours, monotone in float arithmetic too.
__device__ __forceinline__ int zero_bound(int L, int nq, int t) {
  if (t >= nq) return L;
  const float per = (float)L / ((float)nq * (float)(nq + 1));
  return min((int)((float)t * (float)(t + 1) * per), L);
}

// two bf16 in one dword: widen to fp32 (exact), add, round each sum to bf16 (nearest even)
__device__ __forceinline__ uint32_t add_bf16_pairs(uint32_t x, uint32_t o) {
  const float x0 = __uint_as_float(x << 16), x1 = __uint_as_float(x & 0xffff0000u);
  const float o0 = __uint_as_float(o << 16), o1 = __uint_as_float(o & 0xffff0000u);
  bf16x2 s;
  s[0] = (__bf16)(x0 + o0);
  s[1] = (__bf16)(x1 + o1);
  return __builtin_bit_cast(uint32_t, s);
}

__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  bf16x2 v;
  v[0] = (__bf16)lo;
  v[1] = (__bf16)hi;
  return __builtin_bit_cast(uint32_t, v);
}

// Workgroup barrier that waits for this wavefront's LDS traffic only.  __syncthreads() also waits for every outstanding
// global access, the zero rows' stores and the next look-ups among them; the tiles that are loaded into LDS are waited for
// where they have to be (wait_loads).
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// ---- tiles in LDS.  K and V^T tiles go from global memory straight into LDS: no staging registers, no LDS store
// instructions.  Such a load writes the 64 lanes' 16-byte pieces to 1 KiB of consecutive addresses (a block: 8 or 4 rows of
// 128 or 256 bytes), so rows cannot be padded; instead the pieces of a row are stored in an order that depends on the row
// (piece p of row r at position p ^ swizzle, chosen on the global side of the load), and the blocks are kBlock
// bytes apart.  With both, 16 consecutive rows put any one piece into 16 different positions of the 256 bytes that the banks
// cover: row bits 0, 1 (256-byte rows) or 1, 2 (128-byte rows, whose bit 0 selects the half of the 256 bytes) go into
// the low two bits of the position by the exclusive or, the next two (one) through the 64 bytes between blocks.
// A fragment read of k-step i takes piece hi + 2 i: only bit 0 of i meets the swizzle, so two lane offsets and immediates
// reach all of them.
constexpr int kBlock = 1024 + 64;
template <int RB>                                   // bytes of a row: 128 or 256
struct LdsRows {
  static constexpr int LPR = RB / 16, RPB = 64 / LPR;                        // pieces of a row, rows of a block
  __device__ static __forceinline__ int swizzle(int row) { return RB == 256 ? row & 3 : (row >> 1) & 3; }
  // global side: the piece of its row (row lane / LPR of the block) that lane `lane` of a load fetches
  __device__ static __forceinline__ int piece(int lane) { return (lane % LPR) ^ swizzle(lane / LPR); }
  // byte offset of piece hi (+ 2 i: read_off) of row `row`
  __device__ static __forceinline__ int read_base(int row, int hi) { return (row / RPB) * kBlock + (row % RPB) * RB + ((hi ^ swizzle(row)) << 4); }
  __device__ static __forceinline__ int read_off(const int (&base)[2], int i) { return base[i & 1] + 64 * (i >> 1); }
};

// One block: lane l's 16 bytes at (buffer + voff + soff) to LDS byte `lds` + 16 l.  Counted by vmcnt, by nothing the compiler
// tracks: whoever reads the block waits (s_waitcnt vmcnt, then the workgroup barrier) himself.  In assembly because the
// compiler, which cannot tell the slots of a ring apart, would wait for these loads before every fragment read; there is no
// output register that it could reuse while the load is in flight.
// The compiler's hazard pass does not look inside, and a load needs five wait states behind a vector instruction that wrote one
// of its scalar operands (a readfirstlane here, a scalar that comes back from a spill).  PAD: they are in the assembly, whatever
// stands in front of it: for the kernels with block lists, which spill scalars and whose tile numbers come out of a search.
// They cost 0.3 to 0.8 % there (layer under a list 1103 -> 1106 us).  The others hold their operands in scalars that only scalar
// instructions write, and would pay 2.5 % where one long chain is the launch (4 heads x 24071 rows, d = 64, 389 -> 399 us); that
// their assembly is as it should be is tested (test_load_to_lds.py).  m0 is an operand, so that the compiler writes it and
// knows that it did; one wait state in front of the load is due to that.
template <bool PAD>
__device__ __forceinline__ void load_to_lds(u32x4 rsrc, int voff, int soff, int lds) {
#if defined(__HIP_DEVICE_COMPILE__)
  soff = __builtin_amdgcn_readfirstlane(soff);           // (the same in all lanes already; nothing where the compiler knows)
  lds = __builtin_amdgcn_readfirstlane(lds);
  if constexpr (PAD)
    asm volatile("s_nop 4\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"{m0}"(lds), "v"(voff), "s"(rsrc), "s"(soff) : "memory");
  else
    asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"{m0}"(lds), "v"(voff), "s"(rsrc), "s"(soff) : "memory");
#endif
}
// The descriptor of head_rsrc (below) as plain words.
__device__ __forceinline__ u32x4 rsrc_words(const __bf16* base, long long bytes) {
  const unsigned long long p = (unsigned long long)base;
  const auto scalar = [](uint32_t x) -> uint32_t { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); };
  return u32x4{scalar((uint32_t)p), scalar((uint32_t)(p >> 32) & 0xffffu), scalar((uint32_t)bytes), 0x00020000u};
}

// Every load of this wavefront has landed, in registers or in LDS.  The builtin is what the compiler sees; the scheduling
// barriers keep it where it stands.
__device__ __forceinline__ void wait_loads() {
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_waitcnt(0x0F70);                    // vmcnt(0)
  __builtin_amdgcn_sched_barrier(0);
}

// Keys sit in the LDS tile in a permuted row order (bits 2 and 3 of the row swapped), so
// that accumulator register r of lane half hi holds key 16*(r/8) + 8*hi + r%8 of its 32-key
// half tile: the eight probabilities a lane packs for one PV step are then eight CONSECUTIVE
// keys, and the matching V^T operand is one contiguous 16-byte read.
__device__ __forceinline__ int k_row_perm(int lo) { return (lo & ~12) | ((lo & 4) << 1) | ((lo & 8) >> 1); }
__device__ __forceinline__ int key_of(int r, int hi) { return 16 * (r >> 3) + 8 * hi + (r & 7); }

// Key tiles a workgroup visits, in order.  A block list cuts the workgroup's 256 query rows into
// row blocks of `block` tokens (4, 2 or 1 of them); `use` bit j: row block j takes part in the tile
// (they can differ only under a block list; plain causal attention is one row block of 256).
struct Tile {
  int k0;      // first key of the tile, < 0: no more tiles
  int use;
};

struct TileGen {
  const int32_t* list[kMaxLists];   // the lists of the workgroup's row blocks, merged on the fly
  int cnt[kMaxLists], pos[kMaxLists];
  int cur[kMaxLists];               // next unread entry of each list (INT_MAX: exhausted), read one block ahead
  int n_lists, block, tiles_per_block, full;
  int sub, kb, use;
  int plain_n, plain_i;
  bool plain;
  __device__ Tile next() {
    if (plain) {
      if (plain_i >= plain_n) return Tile{-1, 0};
      Tile t{plain_i * BN, 1};
      ++plain_i;
      return t;
    }
    if (sub == 0) {
      // cur[] was read from the lists when the previous block was handed out, at least a tile ago:
      // the look-up is never waited for
      kb = INT_MAX;
#pragma unroll
      for (int j = 0; j < kMaxLists; ++j) kb = min(kb, cur[j]);
      if (kb == INT_MAX) return Tile{-1, 0};
      use = 0;
#pragma unroll
      for (int j = 0; j < kMaxLists; ++j)
        if (cur[j] == kb) {
          use |= 1 << j;
          ++pos[j];
          cur[j] = pos[j] < cnt[j] ? list[j][pos[j]] : INT_MAX;
        }
    }
    const Tile t{kb * block + sub * BN, use};
    sub = sub + 1 == tiles_per_block ? 0 : sub + 1;
    return t;
  }
};

// Entries of a block-list row in front of its first entry outside 0..qb, the whole wavefront together: 64 entries per
// memory round trip (one entry per trip, as a loop over scalar loads runs, is 34 trips at the start of a workgroup for a
// sink and a window of 4096 tokens in blocks of 128).
__device__ __forceinline__ int count_valid(const int32_t* row, int max_blocks, int qb, int lane) {
  for (int base = 0; base < max_blocks; base += 64) {
    const int kb = base + lane < max_blocks ? row[base + lane] : -1;
    const unsigned long long bad = __builtin_amdgcn_ballot_w64(kb < 0 || kb > qb);
    if (bad) return base + __ffsll((long long)bad) - 1;
  }
  return max_blocks;
}

// P^T operand of MFMA k-step hf (16 keys) of a half tile, from the packed probabilities.
__device__ __forceinline__ bf16x8 p_operand(const uint32_t (&pb)[8], int hf) {
  const u32x4 pw = {pb[4 * hf + 0], pb[4 * hf + 1], pb[4 * hf + 2], pb[4 * hf + 3]};
  return __builtin_bit_cast(bf16x8, pw);
}

// Staging of 64-key tiles by NW wavefronts and the reads of their fragments.  Wavefront w loads blocks CH w .. CH w + CH - 1 of
// either tile.  Row R of the K tile in LDS need not be key R: what a lane loads is chosen so that its CH rows are CH
// consecutive keys (one look-up in idx for all of them), and the fragment reads undo that together with k_row_perm.  A
// V^T tile is one contiguous [d][64] block of the tiled tensor.  Offsets that all lanes share go into the scalar offset of
// the load.  Slots of the rings are byte offsets into `smem`.
template <int D, int NW, bool LISTS>
struct Stage {
  using KRows = LdsRows<2 * D>;                   // K tile: [key][d]
  using VRows = LdsRows<2 * BN>;                  // V^T tile: [d][key]
  static constexpr int KHALF = 32 / KRows::RPB * kBlock, VTILE = D / VRows::RPB * kBlock;   // bytes of half a K tile, of a V^T tile
  static constexpr int CH = BN * D / (512 * NW);  // blocks (of 512 elements) of a tile that a wavefront loads
  static constexpr int NS = D / 16, ND = D / 32;  // MFMA k-steps of the QK product, d sub-tiles of the output
  static constexpr int kHalfBlocks = 32 / KRows::RPB, VSUB = 32 / VRows::RPB * kBlock;      // VSUB: bytes between d sub-tiles
  char* smem;
  int row, col;                // keys row .. row + CH - 1 of a K tile, byte in the row
  bool half;                   // (a wavefront's blocks lie in one half tile)
  int lds0, k_lds, v_lds, v_off, v_block;
  int k_rd[2], v_rd[2];
  __device__ __forceinline__ void init(char* smem_, int tid) {
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, lo = lane & 31, hi = lane >> 5;
    smem = smem_;
    lds0 = (int)(uintptr_t)(__attribute__((address_space(3))) char*)smem_;
    row = CH * (tid / KRows::LPR);
    col = 16 * KRows::piece(lane);
    half = wave * CH >= kHalfBlocks;
    k_lds = (wave * CH % kHalfBlocks) * kBlock;
    v_lds = wave * CH * kBlock;
    v_off = (lane / VRows::LPR) * 2 * BN + 16 * VRows::piece(lane);
    v_block = wave * CH * 1024;
    // K operand (A of S^T): MFMA row lo = key k_row_perm(lo) of the half tile, 8 d-values at 8 hi
    constexpr int GR = KRows::RPB * CH;           // keys that a wavefront loads
    const int key = k_row_perm(lo);
    const int at = (key & ~(GR - 1)) | ((key & (CH - 1)) * KRows::RPB) | ((key & (GR - 1)) / CH);
    k_rd[0] = KRows::read_base(at, hi);
    k_rd[1] = k_rd[0] ^ 32;
    // V^T operand (A of O^T): row = d (lo within the 32-row d sub-tile), 8 keys at 8 hi
    v_rd[0] = VRows::read_base(lo, hi);
    v_rd[1] = v_rd[0] ^ 32;
  }
  // row numbers of the K tile at row k0: idx's entries (FUSED) or the rows themselves
  template <bool FUSED>
  __device__ __forceinline__ void look_up(__amdgpu_buffer_rsrc_t idx, int k0, int (&tok)[CH]) const {
    if constexpr (!FUSED) {
#pragma unroll
      for (int i = 0; i < CH; ++i) tok[i] = k0 + row + i;
    } else if constexpr (CH == 4) {
      const u32x4 t = __builtin_amdgcn_raw_buffer_load_b128(idx, row * 4, k0 * 4, 0);
#pragma unroll
      for (int i = 0; i < CH; ++i) tok[i] = t[i];
    } else if constexpr (CH == 2) {
      const u32x2 t = __builtin_amdgcn_raw_buffer_load_b64(idx, row * 4, k0 * 4, 0);
#pragma unroll
      for (int i = 0; i < CH; ++i) tok[i] = t[i];
    } else {
      tok[0] = __builtin_amdgcn_raw_buffer_load_b32(idx, row * 4, k0 * 4, 0);
    }
  }
  // block i of this wavefront's share; row_off: byte offset of the row of K; half0, half1, tile: slots
  __device__ __forceinline__ void load_k(u32x4 K, int row_off, int half0, int half1, int i) const {
    load_to_lds<LISTS>(K, row_off + col, 0, lds0 + (half ? half1 : half0) + k_lds + i * kBlock);
  }
  __device__ __forceinline__ void load_v(u32x4 Vt, int k0, int tile, int i) const {
    load_to_lds<LISTS>(Vt, v_off, k0 * 2 * D + v_block + i * 1024, lds0 + tile + v_lds + i * kBlock);
  }
  __device__ __forceinline__ bf16x8 k_frag(int half_slot, int i) const { return *(const bf16x8*)(smem + half_slot + KRows::read_off(k_rd, i)); }
  // 16 keys from 16 hf on (hf 0 .. 3 over the tile's 64 keys), d sub-tile dt
  __device__ __forceinline__ bf16x8 v_frag(int tile, int hf, int dt) const { return *(const bf16x8*)(smem + tile + VRows::read_off(v_rd, hf) + dt * VSUB); }
  // S^T of a half tile
  template <int QS>
  __device__ __forceinline__ void qk(int half_slot, const bf16x8 (&qf)[QS][NS], f32x16 (&s)[QS]) const {
#pragma unroll
    for (int qs = 0; qs < QS; ++qs) s[qs] = f32x16{0};
#pragma unroll
    for (int st = 0; st < NS; ++st) {
      const bf16x8 kf = k_frag(half_slot, st);
#pragma unroll
      for (int qs = 0; qs < QS; ++qs) s[qs] = mfma32(kf, qf[qs][st], s[qs]);
    }
  }
  // O^T += V^T P^T for half `h` of a tile (two MFMA k-steps of 16 keys)
  template <int QS>
  __device__ __forceinline__ void pv(int tile, int h, const uint32_t (&pb)[QS][8], f32x16 (&o)[QS][ND]) const {
#pragma unroll
    for (int hf = 0; hf < 2; ++hf)
#pragma unroll
      for (int dt = 0; dt < ND; ++dt) {
        const bf16x8 vf = v_frag(tile, 2 * h + hf, dt);
#pragma unroll
        for (int qs = 0; qs < QS; ++qs) o[qs][dt] = mfma32(vf, p_operand(pb[qs], hf), o[qs][dt]);
      }
  }
};

// Row max of one half tile (per query sub-tile), in scaled log2 units.
template <int QS>
__device__ __forceinline__ void row_max(const f32x16 (&s)[QS], float c, float (&mxc)[QS]) {
#pragma unroll
  for (int qs = 0; qs < QS; ++qs) {
    float mx = s[qs][0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[qs][r]);
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    mxc[qs] = mx * c;
  }
}

// Raises the running max (and rescales l, O) only when some row outgrew it by more than kLazy.
template <int ND, int QS>
__device__ __forceinline__ void raise_max(const float (&mxc)[QS], float (&m)[QS], float (&l)[QS], f32x16 (&o)[QS][ND]) {
  bool grow = false;
#pragma unroll
  for (int qs = 0; qs < QS; ++qs) grow = grow || mxc[qs] > m[qs] + kLazy;
  if (__any(grow)) {
#pragma unroll
    for (int qs = 0; qs < QS; ++qs) {
      const float mn = fmaxf(m[qs], mxc[qs]);
      const float alpha = fast_exp2(m[qs] - mn);
      m[qs] = mn;
      l[qs] *= alpha;
#pragma unroll
      for (int dt = 0; dt < ND; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[qs][dt][r] *= alpha;
    }
  }
}

// The same for a half tile held as s * c - m (the form the pipelined iteration keeps between a QK block
// and its exponentials): mx is the row max relative to m.  A raise also shifts the pending half tile.
template <int ND, int QS>
__device__ __forceinline__ void raise_max_rel(const float (&mx)[QS], float (&m)[QS], float (&l)[QS],
                                              f32x16 (&o)[QS][ND], f32x16 (&pending)[QS]) {
  bool grow = false;
#pragma unroll
  for (int qs = 0; qs < QS; ++qs) grow = grow || mx[qs] > kLazy;
  if (__any(grow)) {
#pragma unroll
    for (int qs = 0; qs < QS; ++qs) {
      const float dlt = fmaxf(mx[qs], 0.f);
      const float alpha = fast_exp2(-dlt);
      m[qs] += dlt;
      l[qs] *= alpha;
#pragma unroll
      for (int r = 0; r < 16; ++r) pending[qs][r] -= dlt;
#pragma unroll
      for (int dt = 0; dt < ND; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[qs][dt][r] *= alpha;
    }
  }
}

template <int ND, int QS>
__device__ __forceinline__ void softmax_max(const f32x16 (&s)[QS], float c, float (&m)[QS], float (&l)[QS], f32x16 (&o)[QS][ND]) {
  float mxc[QS];
  row_max<QS>(s, c, mxc);
  raise_max<ND, QS>(mxc, m, l, o);
}

// p = exp2(s*c - m), packed to bf16 pairs in accumulator order; row sums into l.
template <int QS>
__device__ __forceinline__ void softmax_exp(const f32x16 (&s)[QS], float c, const float (&m)[QS], float (&l)[QS], uint32_t (&pb)[QS][8]) {
#pragma unroll
  for (int qs = 0; qs < QS; ++qs) {
    const float mq = m[qs];
    float ps0 = 0.f, ps1 = 0.f;
#pragma unroll
    for (int r = 0; r < 16; r += 2) {
      const float p0 = fast_exp2(fmaf(s[qs][r], c, -mq));
      const float p1 = fast_exp2(fmaf(s[qs][r + 1], c, -mq));
      ps0 += p0;
      ps1 += p1;
      pb[qs][r >> 1] = pack_bf16(p0, p1);
    }
    l[qs] += ps0 + ps1;
  }
}

template <int QS>
__device__ __forceinline__ void mask_half(f32x16 (&s)[QS], int key0, int hi, int qrow0) {
#pragma unroll
  for (int qs = 0; qs < QS; ++qs)
#pragma unroll
    for (int r = 0; r < 16; ++r)
      if (key0 + key_of(r, hi) > qrow0 + 32 * qs) s[qs][r] = -INFINITY;
}

// Output rows of one wavefront: 32 query rows x 32 ND columns from column col0 on.  A lane's accumulator holds four
// consecutive columns of its own row, so storing from the registers would touch 32 rows per instruction, 16 bytes of each;
// the rows change places through LDS of the wavefront's own instead, and leave (and the residual slice arrives) as whole
// rows, 16 bytes per lane, all loads of the slice requested before the first of them is needed (read and written piece by
// piece, the slice took sixteen dependent round trips).  Layer with 28 heads x 16384 of 65536 rows, blocks of 128 and the
// residual stream: 1144 -> 1084 us together with count_valid; dense 32 x 8192: 500 -> 494; 32 x 4096 of 8192: 202.4 -> 199.4.
template <int D, int ND, bool FUSED>
struct RowOut {
  static constexpr int COLS = 32 * ND, LPR = COLS / 8, RPI = 64 / LPR, N = 32 / RPI;   // lanes per row, rows per round, rounds
  static constexpr int RS = 2 * COLS + 16;          // bytes of a row in LDS: the pad walks the rows over all banks
  static constexpr int kLds = 32 * RS;
  int tok[N];                                       // fused: the token of row j RPI + lane / LPR

  __device__ __forceinline__ void look_up(const int32_t* idx_row, int row0, int Lc, int lane) {
    if (FUSED) {
#pragma unroll
      for (int j = 0; j < N; ++j) tok[j] = idx_row[min(row0 + j * RPI + lane / LPR, Lc - 1)];
    }
  }
  // a lane's row, normalised and rounded to bf16, into LDS
  __device__ __forceinline__ void put(const f32x16 (&o)[ND], float inv_l, char* lds, int lane) const {
    const int lo = lane & 31, hi = lane >> 5;
#pragma unroll
    for (int dt = 0; dt < ND; ++dt)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        u32x2 w;
        w[0] = pack_bf16(o[dt][4 * q4 + 0] * inv_l, o[dt][4 * q4 + 1] * inv_l);
        w[1] = pack_bf16(o[dt][4 * q4 + 2] * inv_l, o[dt][4 * q4 + 3] * inv_l);
        *(u32x2*)(lds + lo * RS + 2 * (32 * dt + 8 * q4 + 4 * hi)) = w;
      }
    __builtin_amdgcn_wave_barrier();                // LDS accesses of one wavefront complete in order
  }
  // `between` runs after the loads of the residual slice are requested and before they are needed
  template <typename F>
  __device__ __forceinline__ void store(const AttendArgs& a, int b, int h, int row0, int Lc, int col0, const char* lds, int lane,
                                        F&& between) const {
    const int r0 = row0 + lane / LPR, col = col0 + 8 * (lane % LPR);
    u32x4 x[N];
    __bf16* xh = nullptr;
    if (FUSED && a.X) {
      xh = a.X + ((long long)b * a.L * a.Hq + h) * D + col;
#pragma unroll
      for (int j = 0; j < N; ++j)
        if (r0 + j * RPI < Lc) x[j] = *(const u32x4*)(xh + (long long)tok[j] * a.Hq * D);
    }
    between();
    __bf16* oh = a.O ? a.O + ((long long)b * a.Hq + h) * a.Lc * D + col : nullptr;
    __bf16* fh = FUSED && a.Of ? a.Of + a.os.head(b, h) + col : nullptr;
#pragma unroll
    for (int j = 0; j < N; ++j)
      if (r0 + j * RPI < Lc) {
        const u32x4 w = *(const u32x4*)(lds + (j * RPI + lane / LPR) * RS + 16 * (lane % LPR));
        if (oh) *(u32x4*)(oh + (long long)(r0 + j * RPI) * D) = w;
        if (FUSED && fh) *(u32x4*)(fh + tok[j] * a.os.l) = w;
        if (FUSED && xh) {
          u32x4 y;
#pragma unroll
          for (int i = 0; i < 4; ++i) y[i] = add_bf16_pairs(x[j][i], w[i]);
          *(u32x4*)(xh + (long long)tok[j] * a.Hq * D) = y;
        }
      }
  }
};

// Raw buffer descriptor over one head's rows: loads past `bytes` return zero, so ragged tails
// and tiles beyond the end need no bounds arithmetic in the loop.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t head_rsrc(const __bf16* base, long long bytes) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, (int)bytes, 0x00020000);
}

}  // namespace attend_detail

// attend_split.hip: the 128-row form (launch with a.nq_tiles / a.nk_tiles unset; it sizes its own grid)
hipError_t launch_attend_split(attend_detail::AttendArgs& a, int d, bool fused, hipStream_t st);

}  // namespace tsa
