// Causal attention over the compacted token set (Section 2.2, Stage 1: the attention
// operation on Q^, K^, V^ with cost O(L'^2 d)), also used unchanged as the dense baseline.
//
// Flash-style: one workgroup owns 256 query rows (8 wavefronts x 32 rows, two wavefronts per
// SIMD; a second form: four wavefronts, 128 rows), streams 64-key tiles through LDS (loaded straight into it, in swizzled
// order: LdsRows; K in a ring of three tiles, with four wavefronts of five half tiles, V in a ring of two tiles, one barrier per
// tile), keeps the running max / sum and the output accumulator in registers (online softmax) and never materialises the
// score matrix.
//
// Both products run on v_mfma_f32_32x32x16_bf16 in the TRANSPOSED orientation:
//   S^T = K Q^T   rows = keys, cols = queries  -> a lane owns ONE query of the wavefront's 32
//                 and 32 of the 64 keys of the tile: the row max / row sum of the softmax need
//                 a single cross-lane step (lane <-> lane^32);
//   O^T = V^T P^T rows = d, cols = queries     -> the P^T operand is exactly what the lane
//                 already holds (its query, eight keys per MFMA step): no shuffle and no LDS
//                 round trip for P, and the rescale factor of O is the lane's own.
// V arrives as 64-key transposed tiles ([d][64 keys]) and K rows sit in LDS in a permuted order, so
// that each V^T operand is one 16-byte LDS read holding exactly the eight keys whose probabilities
// the lane has just packed.
// The loop is software-pipelined: the QK product of the next half tile is issued together with
// the softmax arithmetic of the current one, so the matrix pipe and the vector ALU overlap.
// The O rescale is lazy: the running max is only raised when a row's new max exceeds it by
// more than 2^8, so most tiles skip the multiply over the whole accumulator; the final
// division by the row sum makes the result independent of the max actually used.
// The exponent s * scale * log2(e) - m is formed in the PV block that follows a QK block (one fma per
// score, in fp32, in place, next to MFMAs that have little other vector work beside them), so the
// blocks with the exponentials apply exp2 to the half tile as it is; a raise of m in between shifts the
// waiting half tile by the same amount.
// Very short compacted sets (up to 1792 tokens at 32 heads) take the 128-row form of attend_split.hip
// instead (use_split_form below).
// The template is written for QS query sub-tiles per wavefront; QS = 1 is the one that is built.  (QS = 2, 64 rows per wavefront,
// one per SIMD, every LDS fragment feeding two MFMAs, measured slower with the tiles still staged through registers; with
// the loads into LDS it was not timed.  Taking the parameter out gives the fused kernels other registers and costs 1 to
// 1.7 % of their long launches: 32 heads x 16384 rows 2033 -> 2068 us for the layer.)
#include <algorithm>
#include <numeric>

#include "attend_common.h"

namespace tsa {

using namespace attend_detail;

namespace {

// QS = query sub-tiles (of 32 rows) per wavefront, NW = wavefronts per workgroup.  QS = 1: wavefronts of 32 rows, which share
// the SIMD's issue slots (a lone wavefront issues one vector instruction every ~8 clocks, two
// together one every ~5) at the price of one LDS fragment per MFMA.  NW = 8: 256 rows, the two wavefronts of a SIMD
// belong to one workgroup.  NW = 4: 128 rows; the LDS holds two such workgroups (2 x 78336 bytes of 160 KiB, with K
// in a ring of five half tiles instead of three tiles), three at d = 64 (39168 bytes each; 168 VGPRs, of which the fused forms spill 4, with lists 5), which wait
// at their own barriers and start and end one under the other; every K / V tile is staged for half as many rows.
// Which one runs, and what both measured: use_pair_form below.
// LISTS: the launch has a block list.  The plain causal form is a kernel of its own: the look-ups of the tile
// generator would otherwise sit in the tile loop as loads that may be pending, and the compiler's wait for
// them (before it reuses their registers) also waits for the K / V prefetches of the tile just requested.
template <int D, int QS, int NW, bool FUSED, bool LISTS>
__global__ __launch_bounds__(64 * NW, D == 64 && NW == 4 ? 3 : 2 / QS) void attend_kernel(AttendArgs a) {
  constexpr int kThreads = 64 * NW;
  constexpr int RW = 32 * QS;                     // query rows per wavefront
  constexpr int BM = RW * NW;                     // query rows per workgroup
  using Stg = Stage<D, NW, LISTS>;
  constexpr int KHALF = Stg::KHALF, VTILE = Stg::VTILE, CH = Stg::CH;
  constexpr int NS = D / 16;                      // MFMA k-steps of the QK product
  constexpr int ND = D / 32;                      // d sub-tiles of the output
  constexpr int ROWB = D * 2;                     // bytes of one row in global memory
  constexpr int KRING = NW == 8 ? 6 : 5;          // half tiles of the K ring
  __shared__ __attribute__((aligned(1024))) char smem[KRING * KHALF + 2 * VTILE];   // K ring, V ring [2 tiles]

  // ---- workgroup -> (head, query tile).  Consecutive workgroup ids go to different XCDs, so
  // id % 8 picks the XCD; all tiles of a head (and all heads of a KV group) stay on one XCD to
  // share its L2, and the longest (last) query tiles are scheduled first.
  int b, h, from_last;
  workgroup_of(a, blockIdx.x, b, h, from_last);
  // Rows of this batch entry's compacted set: the launch's count, or (fused form with a coverage
  // budget decided on the device) the count read from k_dev; a.Lc stays the capacity, i.e. the row
  // stride of idx and of the tile arrays, and the grid is sized for it.
  int Lc = a.Lc, nq_tiles = a.nq_tiles;
  if (FUSED && a.k_dev) {
    Lc = a.k_dev[b];
    nq_tiles = (Lc + BM - 1) / BM;
  }
  const int qt = nq_tiles - 1 - from_last;
  if (qt < 0) return;
  const long long bh = (long long)b * a.Hq + h;
  const long long bkv = (long long)b * a.kvh + a.by_g.div(h);    // head of K^ / V^ (fused: of the index set and the V tiles)
  // rows of Q and K: the compacted tensors, or (fused) the original ones addressed through idx
  // (fused: row pitch and head offsets come from the caller's layout; byte offsets of a row fit 32 bits
  // and both factors of token * pitch fit 24 bits, checked on the host)
  const int q_pitch = FUSED ? (int)a.qs.l * 2 : ROWB, k_pitch = FUSED ? (int)a.ks.l * 2 : ROWB;
  const __bf16* q_head = FUSED ? a.Q + a.qs.head(b, h) : a.Q + bh * Lc * D;
  const __bf16* k_head = FUSED ? a.K + a.ks.head(b, a.by_g_kv.div(h)) : a.K + bkv * Lc * D;
  const int n_rows = FUSED ? a.L : Lc;
  const __amdgpu_buffer_rsrc_t Qr = head_rsrc(q_head, (long long)n_rows * q_pitch);
  const u32x4 Kr = rsrc_words(k_head, (long long)n_rows * k_pitch);
  const long long vt_bytes = (long long)a.nk_tiles * BN * ROWB;
  const u32x4 Vr = rsrc_words(a.Vt + bkv * (vt_bytes / 2), vt_bytes);
  const int32_t* idx_row = FUSED ? a.idx + bkv * a.Lc : nullptr;
  // index loads past the end of the set return 0 (token 0): such rows are only ever read as keys
  // beyond every query of the workgroup, which causality masks
  const __amdgpu_buffer_rsrc_t Ir = __builtin_amdgcn_make_buffer_rsrc((void*)idx_row, 0, FUSED ? Lc * 4 : 0, 0x00020000);

  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, lo = lane & 31, hi = lane >> 5;
  const int q0 = qt * BM;
  const int wrow0 = q0 + RW * wave;                      // first query row of this wavefront
  const int row_block = LISTS ? a.block : BM;
  const int half_bit = 1 << ((RW * wave) / row_block);   // which row block of the query tile the wavefront is in
  const float c = a.c;
  const float c_ = c;
  const float inv_c = 1.0f / c;                                    // (the chunk loop of the pipelined iteration has its own c)

  // ---- fused form: zero rows of the full-length output.  The workgroup owns a range of the head's
  // tokens (see below) and clears those that inv marks unselected.  The work is
  // spread over the tile loop, one pass of kThreads / (d/8) rows every z_every iterations (the
  // look-up in inv for the next pass is in flight meanwhile), so the stores drain under the compute
  // instead of holding up the start of the workgroup; what is left when the tiles run out is flushed
  // before the epilogue.
  constexpr int LPR = D / 8, ZR = 512 / kThreads, RPT = kThreads / LPR, RPP = ZR * RPT;   // a pass: ZR rows per thread
  const bool zfill = FUSED && a.Of != nullptr;
  const long long o_pitch16 = FUSED ? a.os.l / 8 : LPR;          // 16-byte pieces between rows of the full-length output
  const int32_t* inv_row = nullptr;
  u32x4* zrow = nullptr;
  int z_hi = 0, zt = 0, zr[ZR] = {};                     // end of the range, next rows of this thread, their inv entries
  int z_every = 1, z_count = 1;
  auto start_zero_rows = [&](int n_pipelined) {
    inv_row = a.inv + bkv * a.L;
    // Token range of this workgroup.  Any partition of [0, L) over the query tiles of a head works (a row is
    // cleared iff inv marks it unselected, whoever looks).  The shares grow linearly with the query tile,
    // as the number of tile iterations does, so that every workgroup can clear its share inside its loop.
    const int tok_lo = zero_bound(a.L, nq_tiles, qt);
    z_hi = zero_bound(a.L, nq_tiles, qt + 1);
    zrow = (u32x4*)(a.Of + a.os.head(b, h)) + (tid % LPR);
    zt = tok_lo + tid / LPR;
#pragma unroll
    for (int j = 0; j < ZR; ++j) zr[j] = zt + j * RPT < z_hi ? inv_row[zt + j * RPT] : 0;
    // as evenly over the pipelined iterations as their number allows (RPP is a power of two)
    z_every = max(1, (int)((float)n_pipelined / (float)max(1, (z_hi - tok_lo + RPP - 1) / RPP)));
  };
  auto zero_step = [&]() {
#pragma unroll
    for (int j = 0; j < ZR; ++j)
      if (zr[j] < 0) __builtin_nontemporal_store(u32x4{0u, 0u, 0u, 0u}, zrow + (long long)(zt + j * RPT) * o_pitch16);
    zt += RPP;
#pragma unroll
    for (int j = 0; j < ZR; ++j) zr[j] = zt + j * RPT < z_hi ? inv_row[zt + j * RPT] : 0;
  };

  TileGen gen;
  gen.plain = !LISTS;
  gen.plain_i = 0;
  gen.plain_n = (min(q0 + BM, Lc) + BN - 1) / BN;
  gen.sub = gen.kb = gen.use = 0;
  gen.n_lists = 1;
  gen.block = BM;
  gen.tiles_per_block = BM / BN;
  gen.full = 1;
  int longest_list = 0;
#pragma unroll
  for (int j = 0; j < kMaxLists; ++j) { gen.list[j] = nullptr; gen.cnt[j] = gen.pos[j] = 0; gen.cur[j] = INT_MAX; }
  if (!gen.plain) {
    gen.block = a.block;
    gen.n_lists = max(1, BM / a.block);
    gen.tiles_per_block = a.block / BN;
    gen.full = 0;
    const int nqb = (Lc + a.block - 1) / a.block;
    const int32_t* bl = a.block_list + bh * a.bl_head_stride;
#pragma unroll
    for (int j = 0; j < kMaxLists; ++j) {
      const int qb = q0 / a.block + j;
      if (j < gen.n_lists && qb < nqb) {
        gen.list[j] = bl + (long long)qb * a.max_blocks;
        gen.cnt[j] = count_valid(gen.list[j], a.max_blocks, qb, lane);
        if (gen.cnt[j] > 0) gen.cur[j] = gen.list[j][0];
        gen.full |= 1 << j;
        longest_list = max(longest_list, gen.cnt[j]);
      }
    }
  }

  // ---- staging: global memory -> LDS
  Stg stg;
  stg.init(smem, tid);
  // Rows of the next K tile to be loaded: ktok[i] = row of thread chunk i (fused: the token the
  // compacted row stands for, fetched from idx one tile ahead of the K load that uses it).
  int ktok[CH];
  auto row_off = [&](int tok) -> int { return FUSED ? (int)__umul24(tok, k_pitch) : tok * ROWB; };
  auto fetch_tok = [&](int k0, int (&tok)[CH]) { stg.template look_up<FUSED>(Ir, k0, tok); };
  auto load_k = [&](const int (&tok)[CH], int half0, int half1, int i) { stg.load_k(Kr, row_off(tok[i]), half0, half1, i); };
  auto load_v = [&](int k0, int tile, int i) { stg.load_v(Vr, k0, tile, i); };

  f32x16 o[QS][ND];
  float m[QS], l[QS];
#pragma unroll
  for (int qs = 0; qs < QS; ++qs) {
    m[qs] = kNegBig;
    l[qs] = 0.f;
#pragma unroll
    for (int dt = 0; dt < ND; ++dt) o[qs][dt] = f32x16{0};
  }

  // Ring slots (byte offsets).  K half tiles: kh(0) = K(t) half 1, kh(1) and kh(2) = K(t+1), K(t+2) goes to kh(3) and kh(4)
  // (whose last readers were in iteration t - 1); V tiles: V(t) in vc, V(t+1) goes to vn.  With eight wavefronts the
  // LDS has room for three whole tiles, whose halves are one offset apart (0.4 % of a long launch).
  int kr[5];
#pragma unroll
  for (int j = 0; j < 5; ++j) kr[j] = (NW == 8 ? 2 * j : j) * KHALF;   // (eight wavefronts: tiles t, t + 1, t + 2)
  auto kh = [&](int j) -> int { return NW == 8 ? kr[(j + 1) >> 1] + ((j + 1) & 1) * KHALF : kr[j]; };
  auto k_first = [&]() -> int { return NW == 8 ? kr[0] : kr[3]; };         // K(0) half 0, read by the prologue alone
  int vc = KRING * KHALF;
  int vn = KRING * KHALF + VTILE;
  auto rotate = [&]() {
    int t0 = kr[0], t1 = kr[1];
    if (NW == 8) { kr[0] = kr[1]; kr[1] = kr[2]; kr[2] = t0; }
    else { kr[0] = kr[2]; kr[1] = kr[3]; kr[2] = kr[4]; kr[3] = t0; kr[4] = t1; }
    t0 = vc; vc = vn; vn = t0;
  };

  // ---- prologue
  Tile T0 = gen.next(), T1 = gen.next(), T2 = gen.next();
  f32x16 sA[QS], sB[QS];
  uint32_t pA[QS][8], pB[QS][8];
  bf16x8 qf[QS][NS];             // Q^T operand fragments, in registers for the whole kernel
  {
    // Everything the first iteration needs is requested in two rounds, first the look-ups, then the
    // rows they name and V: two memory latencies instead of six (0.5 to 1 % of a launch up to 32 x 16384 rows).  Tiles that do not exist are
    // replaced by tile 0: loaded, never used.
    int qtok[QS], k0tok[CH], k1tok[CH];
#pragma unroll
    for (int qs = 0; qs < QS; ++qs) {
      const int qr = wrow0 + 32 * qs + lo;
      qtok[qs] = FUSED ? __builtin_amdgcn_raw_buffer_load_b32(Ir, qr * 4, 0, 0) : qr;
    }
    fetch_tok(max(T0.k0, 0), k0tok);
    fetch_tok(max(T1.k0, 0), k1tok);
    fetch_tok(max(T2.k0, 0), ktok);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < CH; ++i) load_k(k0tok, k_first(), kh(0), i);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int qs = 0; qs < QS; ++qs) {
      const int qr = wrow0 + 32 * qs + lo;
      int qrow_off = qr * ROWB;
      if (FUSED) qrow_off = qr < Lc ? (int)__umul24(qtok[qs], q_pitch) : a.L * q_pitch;   // past the end: out of the buffer's range, reads zeros
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(Qr, qrow_off + 16 * hi + 32 * s, 0, 0);
        qf[qs][s] = __builtin_bit_cast(bf16x8, v);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < CH; ++i) load_k(k1tok, kh(1), kh(2), i);
#pragma unroll
    for (int i = 0; i < CH; ++i) load_v(max(T0.k0, 0), vc, i);
  }
  // (the zero rows' first look-ups while those are under way)
  if (zfill) start_zero_rows(gen.plain ? q0 / BN - 1 : gen.tiles_per_block * longest_list - 6);
  // Everything has landed (the next wait for loads is at the end of the first iteration; and the compiler must know that the
  // Q fragments and look-ups have, or it would carry them as "possibly pending" into the loop).
  wait_loads();
  lds_barrier();
  if (T0.k0 >= 0) stg.template qk<QS>(k_first(), qf, sA);
  if (NW != 8) lds_barrier();                            // that slot is written in the first iteration
  auto wave_active = [&](const Tile& t) -> bool { return t.k0 >= 0 && (t.use & half_bit) && t.k0 <= wrow0 + RW - 1; };
  if (wave_active(T0)) {
    if (T0.k0 + 31 > wrow0) mask_half<QS>(sA, T0.k0, hi, wrow0 + lo);
    softmax_max<ND, QS>(sA, c, m, l, o);
  }

  // Invariant at the top of an iteration: sA = S^T of the first half of tile T0, already masked
  // and already covered by the running max m (if this wavefront takes part in T0); K(T0)'s second half in
  // kh(0), K(T1) in kh(1) and kh(2), V(T0) in vc, nothing in flight; ktok = rows of T2.  The iteration requests K(T2) and V(T1)
  // at its start (the slots' last readers are behind the barrier) and waits for them at its end.
  //
  // Order inside an iteration: every block of 16 MFMAs is issued next to vector work that does
  // not depend on it, so the matrix pipe and the VALU overlap within the wavefront:
  //   QK(T0, half 1)      with  exp(sA)
  //   PV(T0, half 0)      with  max(sB)            [then the rare raise of m, rescale of O]
  //   QK(T1, half 0)      with  exp(sB)
  //   PV(T0, half 1)      with  max(sA of T1)            [then the rare raise of m]

  // ---- the pipelined iteration: one key tile that lies entirely below the workgroup's first
  // row and is used by all its wavefronts (as is the tile after it) needs no mask and no
  // per-wavefront decisions; loads past the end return zeros, so nothing in it is conditional
  // except the rare raise of the running max.
  // The iteration is a stream of 32 chunks of two MFMAs each:
  //    0.. 7  S^T(T0, half 1) -> sB      with  exp(sA) -> pA
  //    8..15  O^T += V^T(T0, half 0) pA  with  row max of sB          [then the rare raise of m]
  //   16..23  S^T(T1, half 0) -> sA      with  exp(sB) -> pB
  //   24..31  O^T += V^T(T0, half 1) pB  with  row max of sA         [wait for the tiles requested, barrier, rare raise of m]
  // Inside this loop sA and sB hold s * c - m by the time their exponentials are due (formed by an fma
  // per element in the PV block after the chain), so the
  // exponent is the register itself and the row max is relative to m; a raise of m between the two shifts
  // the pending half tile by the same amount.
  // Each chunk consumes one 16-byte LDS fragment per lane (a K fragment or a V^T fragment);
  // fragments are fetched kPF chunks ahead through a small register ring that runs across the
  // blocks and across iterations, so the LDS latency is hidden.
  constexpr int kPF = TSA_PF, kRing = TSA_RING, kChunks = 4 * NS;
  static_assert(NS == 8 || NS == 4, "chunk stream is laid out for d = 128 or 64");
  constexpr int CPB = kChunks / 4;                       // chunks per block
  // slot = chunk % kRing must mean the same slot in consecutive iterations; a fragment must not be
  // overwritten before it is consumed; and the fragments fetched across the iteration boundary
  // must all belong to block 0 (K of the next tile, complete since the previous barrier), not to
  // the V tile that is still arriving during this iteration
  static_assert(kChunks % kRing == 0 && kRing > kPF && kPF <= CPB, "fragment ring does not fit the chunk stream");
  bf16x8 kfr[kRing];
  // fragment fetch for chunk c of the iteration whose half tiles of K and tile of V sit in (k1_, k2_, vc_)
  auto fetch = [&](int c, int k1_, int k2_, int vc_) {
    const int blk = c / CPB, i = c % CPB, slot = c % kRing;
    if (blk == 0) kfr[slot] = stg.k_frag(k1_, i);
    else if (blk == 2) kfr[slot] = stg.k_frag(k2_, i);
    else kfr[slot] = stg.v_frag(vc_, (blk == 3 ? 2 : 0) + i / ND, i % ND);
  };
  auto prime_ring = [&]() {
#pragma unroll
    for (int c = 0; c < kPF; ++c) fetch(c, kh(0), kh(1), vc);
  };
  // v1: first key of the V tile to load (tile T1); tok3: first compacted row of the K tile whose rows are looked up (tile T3)
  auto fast_iter = [&](const int v1, const int tok3) {
    float mxc[QS], mx[QS], ps0[QS], ps1[QS];
    f32x16 acc[QS];
#pragma unroll
    for (int c = 0; c < kChunks; ++c) {
      const int blk = c / CPB, i = c % CPB, slot = c % kRing;
      // A wavefront in a block with exponentials has the longer chain of vector instructions between
      // its MFMAs: it takes precedence over the other wavefront of its SIMD while it is there
      // (measured: 3 % faster on random values, 5 % on zeros, against equal priorities).
      if (i == 0) {
        if (blk == 0 || blk == 2) __builtin_amdgcn_s_setprio(2);
        else __builtin_amdgcn_s_setprio(0);
      }
      // prefetch kPF chunks ahead; the first chunks of the next iteration read the rotated slots
      if (c + kPF < kChunks) fetch(c + kPF, kh(0), kh(1), vc);
      else fetch(c + kPF - kChunks, kh(2), kh(3), vn);
      // K(t+2) -> kh(3), kh(4), V(t+1) -> vn, then the look-ups of the K tile after that
      if (c < CH) load_k(ktok, kh(3), kh(4), c);
      else if (c < 2 * CH) load_v(v1, vn, c - CH);
      else if (c == 2 * CH) fetch_tok(tok3, ktok);
      if (blk == 0 || blk == 2) {
        const f32x16 (&s_in)[QS] = blk == 0 ? sA : sB;
        uint32_t (&p_out)[QS][8] = blk == 0 ? pA : pB;
        constexpr int EPS = 16 / NS;
        // one MFMA, then the exponentials of one query sub-tile: the vector work runs in the
        // shadow of the MFMA that was just issued
#pragma unroll
        for (int qs = 0; qs < QS; ++qs) {
          if (i == 0) acc[qs] = f32x16{0};
          acc[qs] = mfma32(kfr[slot], qf[qs][i], acc[qs]);
#pragma unroll
          for (int e = 0; e < EPS; e += 2) {
            const int r = EPS * i + e;
            const float p0 = fast_exp2(s_in[qs][r]);
            const float p1 = fast_exp2(s_in[qs][r + 1]);
            if (r == 0) { ps0[qs] = p0; ps1[qs] = p1; }
            else { ps0[qs] += p0; ps1[qs] += p1; }
            p_out[qs][r >> 1] = pack_bf16(p0, p1);
          }
          if (qs + 1 < QS) __builtin_amdgcn_sched_barrier(0);
        }
        if (i == CPB - 1) {
          f32x16 (&s_out)[QS] = blk == 0 ? sB : sA;
#pragma unroll
          for (int qs = 0; qs < QS; ++qs) {
            s_out[qs] = acc[qs];
            l[qs] += ps0[qs] + ps1[qs];
          }
        }
      } else {
        f32x16 (&s_in)[QS] = blk == 1 ? sB : sA;
        const uint32_t (&pb)[QS][8] = blk == 1 ? pA : pB;
        const int hf = i / ND, dt = i % ND;
        constexpr int EPC = 16 / CPB;
        const bf16x8 vf = kfr[slot];
#pragma unroll
        for (int qs = 0; qs < QS; ++qs) {
          o[qs][dt] = mfma32(vf, p_operand(pb[qs], hf), o[qs][dt]);
          // the half tile that the last QK block left as plain scores becomes s * c - m here, two elements
          // per chunk, next to the MFMAs of a PV block that has little else to do
#pragma unroll
          for (int e = 0; e < EPC; ++e) s_in[qs][EPC * i + e] = fmaf(s_in[qs][EPC * i + e], c_, -m[qs]);
          if (i == 0) mx[qs] = s_in[qs][0];
          if (EPC == 2) mx[qs] = __builtin_fmaxf(__builtin_fmaxf(mx[qs], s_in[qs][2 * i]), s_in[qs][2 * i + 1]);
          else {
#pragma unroll
            for (int e = 0; e < EPC; ++e) mx[qs] = fmaxf(mx[qs], s_in[qs][EPC * i + e]);
          }
          if (qs + 1 < QS) __builtin_amdgcn_sched_barrier(0);
        }
        if (i == CPB - 1) {
#pragma unroll
          for (int qs = 0; qs < QS; ++qs) mxc[qs] = fmaxf(mx[qs], __shfl_xor(mx[qs], 32));
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      if (c == 2 * CPB - 1) {
        raise_max_rel<ND, QS>(mxc, m, l, o, sB);
      }
    }
    wait_loads();
    // (behind the wait: the next one comes an iteration later, when the stores have long been acknowledged)
    if (FUSED && zfill && --z_count <= 0) {
      zero_step();
      z_count = z_every;
    }
    lds_barrier();
    raise_max_rel<ND, QS>(mxc, m, l, o, sA);
    rotate();
  };

  // ---- tile loop.  A tile takes the pipelined iteration when it and the tile after it lie below
  // the workgroup's first row and are used by both halves of the workgroup (plain causal: every
  // tile but the last five; sink + window lists: all but the first and last few); diagonal tiles,
  // tiles only one half visits and the tile in front of either take the general iteration, with
  // masks and per-wavefront decisions.  Both keep the same invariant, so they alternate freely.
  auto pipelined = [&](const Tile& t) -> bool { return t.k0 >= 0 && t.use == gen.full && t.k0 + BN <= q0; };
  while (T0.k0 >= 0) {
    if (pipelined(T0) && pipelined(T1)) {
      // the pipelined iterations hold their half tiles as s * c - m: sA enters and leaves in that form
#pragma unroll
      for (int qs = 0; qs < QS; ++qs)
#pragma unroll
        for (int r = 0; r < 16; ++r) sA[qs][r] = fmaf(sA[qs][r], c_, -m[qs]);
      prime_ring();
      do {
        const Tile T3 = gen.next();
        // tiles that do not exist are replaced by tile 0 in the prefetches: loaded, never used
        fast_iter(max(T1.k0, 0), max(T3.k0, 0));
        T0 = T1; T1 = T2; T2 = T3;
      } while (pipelined(T0) && pipelined(T1));
      if (T0.k0 < 0) break;
#pragma unroll
      for (int qs = 0; qs < QS; ++qs)
#pragma unroll
        for (int r = 0; r < 16; ++r) sA[qs][r] = (sA[qs][r] + m[qs]) * inv_c;
    }
    const Tile T3 = gen.next();
#pragma unroll
    for (int i = 0; i < CH; ++i) {
      if (T2.k0 >= 0) load_k(ktok, kh(3), kh(4), i);
      if (T1.k0 >= 0) load_v(T1.k0, vn, i);
    }
    if (T3.k0 >= 0) fetch_tok(T3.k0, ktok);
    // A wavefront computes what its rows see and nothing else: the others of its SIMD need the matrix pipe.  (Every product of
    // every tile by every wavefront: 32 heads x 8192 rows 476 us instead of 470, x 4096 133 instead of 131, 64 x 2401 with four wavefronts
    // 111.3 instead of 110.1.)
    if (wave_active(T0)) {
      const bool second = T0.k0 + 32 <= wrow0 + RW - 1;    // some row of the wavefront sees the second half
      if (second) stg.template qk<QS>(kh(0), qf, sB);
      softmax_exp<QS>(sA, c, m, l, pA);
      stg.template pv<QS>(vc, 0, pA, o);
      if (second) {
        if (T0.k0 + BN - 1 > wrow0) mask_half<QS>(sB, T0.k0 + 32, hi, wrow0 + lo);
        softmax_max<ND, QS>(sB, c, m, l, o);
        softmax_exp<QS>(sB, c, m, l, pB);
        stg.template pv<QS>(vc, 1, pB, o);
      }
    }
    if (wave_active(T1)) {
      stg.template qk<QS>(kh(1), qf, sA);
      if (T1.k0 + 31 > wrow0) mask_half<QS>(sA, T1.k0, hi, wrow0 + lo);
      softmax_max<ND, QS>(sA, c, m, l, o);
    }
    wait_loads();
    lds_barrier();
    T0 = T1; T1 = T2; T2 = T3;
    rotate();
  }

  // ---- fused form: the zero rows the tile loop did not get to
  auto flush_zero_rows = [&]() {
    // Latency-bound: a batch of look-ups is a memory round trip.  Sixteen rows per thread and batch, the
    // look-ups of the next batch requested before the stores of the current one (so that waiting for them
    // never includes waiting for those stores to be acknowledged).
    constexpr int kBatch = 16;
#pragma unroll
    for (int j = 0; j < ZR; ++j)
      if (zr[j] < 0) __builtin_nontemporal_store(u32x4{0u, 0u, 0u, 0u}, zrow + (long long)(zt + j * RPT) * o_pitch16);
    int t0 = zt + RPP;
    int r[kBatch];
#pragma unroll
    for (int j = 0; j < kBatch; ++j) r[j] = t0 + j * RPT < z_hi ? inv_row[t0 + j * RPT] : 0;
    while (t0 < z_hi) {
      const int t1 = t0 + kBatch * RPT;
      int rn[kBatch];
#pragma unroll
      for (int j = 0; j < kBatch; ++j) rn[j] = t1 + j * RPT < z_hi ? inv_row[t1 + j * RPT] : 0;
#pragma unroll
      for (int j = 0; j < kBatch; ++j)
        if (r[j] < 0) __builtin_nontemporal_store(u32x4{0u, 0u, 0u, 0u}, zrow + (long long)(t0 + j * RPT) * o_pitch16);
#pragma unroll
      for (int j = 0; j < kBatch; ++j) r[j] = rn[j];
      t0 = t1;
    }
  };

  // ---- epilogue: normalise, round to bf16, store the rows (RowOut).  The LDS is free: every wavefront is past the
  // barrier behind the last read of a tile.
  using Out = RowOut<D, ND, FUSED>;
  static_assert(NW * Out::kLds <= KRING * KHALF + 2 * VTILE, "the rows of all wavefronts fit the tile rings");
  char* const lds_out = smem + wave * Out::kLds;
#pragma unroll
  for (int qs = 0; qs < QS; ++qs) {
    const int row0 = wrow0 + 32 * qs;
    const float lt = l[qs] + __shfl_xor(l[qs], 32);
    const float inv_l = lt > 0.f ? 1.0f / lt : 0.f;
    Out out;
    out.look_up(idx_row, row0, Lc, lane);
    out.put(o[qs], inv_l, lds_out, lane);
    out.store(a, b, h, row0, Lc, 0, lds_out, lane, [&]() { if (zfill && qs == 0) flush_zero_rows(); });
    if (a.lse && hi == 0 && row0 + lo < Lc) a.lse[bh * a.Lc + row0 + lo] = (m[qs] + log2f(lt)) * kLn2;
  }
}

}  // namespace

namespace {

// Which form runs: 0 = chosen per launch, 1 = always 256 rows per workgroup, 2 = always 128 rows with
// the keys split over two groups of wavefronts, 3 = always 128 rows with four wavefronts (measurement
// support: set_attend_form).
int g_attend_form = 0;

// Longest chain of a launch (the last query tile of a head: 4 nq tiles of 64 keys for nq tiles of 256 rows) over
// the work the chip has per CU (BH * 2 nq (nq + 1) tile steps over 256 CUs).
double chain_ratio(const AttendArgs& a) {
  const long long nq = (a.Lc + BM - 1) / BM;
  return 512.0 / (double)(a.BH * (nq + 1));
}

// The split form pays where the longest chain and not the chip's throughput is the launch: it halves that chain, and stages
// every K / V tile for half as many rows and half as many keys per wavefront.  The ratio from which it does rises with
// the number of heads: the more heads, the fewer rows at the same ratio, and the more the start and the merge of its
// workgroups weigh.  us of the launch, fused, d = 128, split / four wavefronts / 256 rows: 4 heads x 18894 rows (ratio 1.71) 391 / 410 / 436,
// x 20942 (1.54) 469 / 480 / 503 (below the line, which is 1.57 for 4 heads: 2 % given away to one line for all); 8 x 9422 (1.68)
// 205 / 211 / 227, x 9934 (1.60) 225 / 226 / 242; 16 x 4046 (1.88) 86 / 91 / 101, x 4302 (1.78) 96 / 98 / 108;
// 20 x 3278 (1.83) 77.7 / 77.0 / 84.7; 32 x 901 (3.2) 22.0 / 23.4 / 30.5, x 1742 (2.0) 43.1 / 44.8 / 49.4 (at d = 64 31.1 / 32.6 / 36.9,
// plain x 1792 28.7 / 31.8); 40 x 1250 (2.13) 35.1 / 34.0 / 38.6; 64 x 738 (2.0) 28.1 / 24.8 / 28.0.  One rule for
// tsa_attend on compacted tensors and the fused launch keeps tsa_forward and the separate calls the same bit for bit.
// Under a block list the windows bound the chains, and how long they are only the device knows: a row of the list may be
// mostly -1, so its room for entries says nothing.  The form is taken where it is the faster one for every window, which is
// while all of its workgroups run at once, one per CU.  Split / four wavefronts / 256 rows, us, fused with a residual stream, rows of the
// list with room for the whole set: 8 heads x 4096 rows, d = 128, (256 workgroups) window 256, blocks of 64 25.4 / 27.5 / 35.1,
// of 128 24.1 / 26.8 / 34.1; whole set 78.9 / 92.3 / 118.2 and 71.3 / 87.0 / 106.7; 64 x 512, blocks of 64, window 64 and whole set: 0.90 and 0.93 of
// four wavefronts.  With more workgroups it loses on short windows what it gains on long ones: 12 x 4096 (384), blocks of 64, 256 44.2 / 31.9 /
// 35.9, 1024 67.3 / 49.3 / 54.6, 2048 76.9 / 67.2 / 79.1, whole set 82.1 / 95.9 / 118.9; 16 x 4096 (512), blocks of 128, 2048 88.0 / 73.4 / 74.8, whole
// set 93.2 / 100.1 / 108.6.
// Blocks of 64 take it only under rows with room for the whole set, and count the workgroups without a tile too: where a head's
// tiles do not divide evenly into its parts (map_workgroups), those hold CUs back (12 x 2600, 252 workgroups in a grid of 264, blocks of
// 64, window 128: 30.8 / 24.6 / 30.3).  Blocks of 128 and more go by the workgroups that have one: in such a grid the form is
// faster on long windows (12 x 2600, blocks of 128, 2688 51.6 / 62.3 / 72.0) and slower on short ones (128 30.1 / 24.3 / 30.0).
bool use_split_form(const AttendArgs& a) {
  if (g_attend_form) return g_attend_form == 2;
  if (!a.block_list) return chain_ratio(a) >= (a.BH <= 32 ? std::min(1.5 + 0.0175 * a.BH, 2.0) : 1.5 + 0.0175 * a.BH);
  const bool small_blocks = a.block < 128;
  if (small_blocks && (long long)a.max_blocks * a.block < a.Lc) return false;
  const int nq = (a.Lc + 127) / 128, parts = small_blocks ? 8 / std::gcd(a.BH, 8) : 1;
  return (long long)a.BH * parts * ((nq + parts - 1) / parts) <= 256 && chain_ratio(a) >= 1.8;
}

// Four wavefronts per workgroup (two or three workgroups per CU) against 256 rows, us of the fused launch:
//   d = 64 (three wavefronts per SIMD instead of two): 32 heads x 4096 rows 88.0 / 87.4, x 8192 313 / 319, x 16384
//     1180 / 1223, 96 x 1500 48.2 / 53.2, sink + window lists 28 x 16384 527 / 568 (blocks of 256), 518 / 596 (128): always.  (Just above
//     768 workgroups a second, nearly empty round costs 5 %: 12 x 9000 167 / 158; 32 x 3277 66.4 / 63.0.)
//   d = 128, block lists with blocks of 64 or 128: a workgroup walks the lists of one or two row blocks instead of the
//     union of up to four, which counts where the window is short: 28 x 16384 with a window of 1024 333 / 371 (blocks of 64), 340 / 378 (128),
//     of 4096 with the residual stream 881 / 894 (64), 862 / 854 (128), 28 x 4096, 1024, 84.5 / 98.8 (64); with blocks of 256
//     only for few heads, by the ratio below.
//   d = 128, plain: a start and an end hidden under the other workgroup are worth more than the second staging of
//     the tiles as long as the chains are short: 128 heads x 600 rows 30.7 / 37.2, 96 x 1000 43.4 / 44.1, 64 x 1500 52.4 / 52.0,
//     32 x 2500 67.5 / 72.3, 96 x 2400 163 / 174, 40 x 3000 105.5 / 104.2, 32 x 3277 109 / 109, 64 x 3300 189 / 189; 32 x 3500 113 / 111,
//     64 x 4000 289 / 275, 32 x 8192 521 / 504, x 32768 8090 / 7750; and where few heads leave the longest chain
//     in charge (16 x 5000 122 / 131, ratio 1.52).
constexpr int kPairRows = 3328;

bool use_pair_form(const AttendArgs& a, int d) {
  if (g_attend_form) return g_attend_form == 3;
  return d == 64 || (a.block_list && a.block < 256) || (!a.block_list && a.Lc <= kPairRows) || chain_ratio(a) >= 1.3;
}

template <bool FUSED, int NW>
hipError_t launch_rows(AttendArgs& a, int d, hipStream_t st) {
  constexpr int rows = 32 * kQS * NW;
  a.nq_tiles = (a.Lc + rows - 1) / rows;
  a.nk_tiles = (a.Lc + BN - 1) / BN;
  map_workgroups(a);
  const unsigned grid = grid_for(a);
  if (a.block_list) {
    if (d == 128) attend_kernel<128, kQS, NW, FUSED, true><<<grid, 64 * NW, 0, st>>>(a);
    else attend_kernel<64, kQS, NW, FUSED, true><<<grid, 64 * NW, 0, st>>>(a);
  } else {
    if (d == 128) attend_kernel<128, kQS, NW, FUSED, false><<<grid, 64 * NW, 0, st>>>(a);
    else attend_kernel<64, kQS, NW, FUSED, false><<<grid, 64 * NW, 0, st>>>(a);
  }
  return hipGetLastError();
}

template <bool FUSED>
hipError_t launch_any(AttendArgs& a, int d, hipStream_t st) {
  if (kQS == 1 && use_split_form(a)) return launch_attend_split(a, d, FUSED, st);
  if (kQS == 1 && use_pair_form(a, d)) return launch_rows<FUSED, 4>(a, d, st);
  return launch_rows<FUSED, 8 / kQS>(a, d, st);
}

}  // namespace

void set_attend_form(int form) { g_attend_form = form; }

hipError_t launch_attend(int B, int Hq, int kv_heads, int Lc, int d, float scale, const void* Qc, const void* Kc,
                         const void* Vt, const int32_t* block_list, int block_size, int max_blocks_per_row,
                         int block_list_per_head, void* Oc, float* lse, hipStream_t st) {
  AttendArgs a;
  a.block = block_list ? block_size : BM;
  a.bl_head_stride = block_list_per_head ? (long long)((Lc + a.block - 1) / a.block) * max_blocks_per_row : 0;
  a.Q = (const __bf16*)Qc; a.K = (const __bf16*)Kc; a.Vt = (const __bf16*)Vt; a.O = (__bf16*)Oc;
  a.lse = lse; a.block_list = block_list; a.max_blocks = max_blocks_per_row;
  a.BH = B * Hq; a.Hq = Hq; a.kvh = kv_heads; a.Lc = Lc;
  a.c = scale * kLog2e;
  a.idx = nullptr; a.inv = nullptr; a.Of = nullptr; a.X = nullptr; a.L = Lc; a.Hkv = kv_heads;
  a.k_dev = nullptr;
  a.qs = a.ks = a.os = Strides{0, 0, 0};
  return launch_any<false>(a, d, st);
}

hipError_t launch_attend_fused(const Dims& dm, const void* Q, const void* K, const void* Vt, const int32_t* idx,
                               const int32_t* inv, int k_keep, const int32_t* block_list, int block_size,
                               int max_blocks_per_row, void* Oc, void* O, void* residual, hipStream_t st,
                               const int32_t* k_dev) {
  AttendArgs a;
  a.k_dev = k_dev;
  a.qs = dm.q; a.ks = dm.kv; a.os = dm.o;
  a.block = block_list ? block_size : BM;
  a.Q = (const __bf16*)Q; a.K = (const __bf16*)K; a.Vt = (const __bf16*)Vt; a.O = (__bf16*)Oc;
  a.lse = nullptr; a.block_list = block_list; a.max_blocks = max_blocks_per_row;
  a.bl_head_stride = dm.block_list_per_head ? (long long)((k_keep + a.block - 1) / a.block) * max_blocks_per_row : 0;
  a.BH = dm.B * dm.Hq; a.Hq = dm.Hq; a.kvh = dm.group_mode ? dm.Hkv : dm.Hq; a.Lc = k_keep;
  a.c = dm.scale * kLog2e;
  a.idx = idx; a.inv = inv; a.Of = (__bf16*)O; a.X = (__bf16*)residual; a.L = dm.L; a.Hkv = dm.Hkv;
  return launch_any<true>(a, dm.d, st);
}

}  // namespace tsa
