// Causal attention over the compacted token set (Section 2.2, Stage 1), the form for VERY SHORT sets
// (a couple of thousand compacted tokens): one workgroup owns 128 query rows, and its eight
// wavefronts are four row groups (32 rows) x two key groups: of every 64-key tile, key group 0 takes
// keys 0..31 and key group 1 keys 32..63, each with its own running max / sum / output accumulator;
// the two partial results of a row group are merged once, at the end, through LDS.
//
// Why: a wavefront walks its key tiles one after the other, so the time of a launch cannot fall
// below the longest chain (the last query tile of a head).  With 256 rows per workgroup and a few
// thousand compacted tokens that chain, not the chip's throughput, is the makespan.  Splitting the
// keys of a tile over two wavefronts halves the chain per row (a workgroup finishes 128 keys per
// iteration instead of 64) and doubles the number of workgroups, at the price of staging every K / V
// tile for 128 instead of 256 rows.
//
// The iteration is the one of the 256-row kernel (attend.hip): per wavefront a stream of 32 chunks,
//    S^T(half 1) with exp(half 0) | PV(half 0) with the row max of half 1 | S^T(next half 0) with
//    exp(half 1) | PV(half 1) with the row max of the next half 0,
// where "half 0 / half 1" of an iteration are the wavefront's 32 keys of the step's first / second
// tile: one step = two 64-key tiles (a, b) = 128 keys, one barrier per step.
// LDS: K tiles of three steps are resident (ring of five tiles: b of the current step, a and b of the
// next one readable, a and b of the step after arriving), V tiles of two steps (ring of four): the tiles go straight into
// LDS (Stage), and the fragments an iteration reads ahead across its closing barrier arrived an iteration earlier.
#include "attend_common.h"

#include <type_traits>

namespace tsa {

using namespace attend_detail;

namespace {

constexpr int BMS = 128;                // query rows per workgroup
constexpr int kThreadsS = 512;

struct Step {
  Tile a, b;                            // the two 64-key tiles of a step; b.k0 < 0: the step has one tile
};

// LISTS: the launch has a block list (a kernel of its own, see attend.hip)
template <int D, bool FUSED, bool LISTS>
__global__ __launch_bounds__(kThreadsS, 2) void attend_split_kernel(AttendArgs a) {
  constexpr int QS = 1;
  constexpr int kThreads = kThreadsS;
  constexpr int RW = 32;
  using Stg = Stage<D, kThreads / 64, LISTS>;
  constexpr int KHALF = Stg::KHALF, KTILE = 2 * KHALF, VTILE = Stg::VTILE, CH = Stg::CH;
  constexpr int NS = D / 16;
  constexpr int ND = D / 32;
  constexpr int ROWB = D * 2;
  constexpr int NKT = 5, NVT = 4;                 // ring slots
  __shared__ __attribute__((aligned(1024))) char smem[NKT * KTILE + NVT * VTILE];

  int b, h, from_last;
  workgroup_of(a, blockIdx.x, b, h, from_last);
  int Lc = a.Lc, nq_tiles = a.nq_tiles;
  if (FUSED && a.k_dev) {
    Lc = a.k_dev[b];
    nq_tiles = (Lc + BMS - 1) / BMS;
  }
  const int qt = nq_tiles - 1 - from_last;
  if (qt < 0) return;
  const long long bh = (long long)b * a.Hq + h;
  const long long bkv = (long long)b * a.kvh + a.by_g.div(h);
  const int q_pitch = FUSED ? (int)a.qs.l * 2 : ROWB, k_pitch = FUSED ? (int)a.ks.l * 2 : ROWB;
  const __bf16* q_head = FUSED ? a.Q + a.qs.head(b, h) : a.Q + bh * Lc * D;
  const __bf16* k_head = FUSED ? a.K + a.ks.head(b, a.by_g_kv.div(h)) : a.K + bkv * Lc * D;
  const int n_rows = FUSED ? a.L : Lc;
  const __amdgpu_buffer_rsrc_t Qr = head_rsrc(q_head, (long long)n_rows * q_pitch);
  const u32x4 Kr = rsrc_words(k_head, (long long)n_rows * k_pitch);
  const long long vt_bytes = (long long)a.nk_tiles * BN * ROWB;
  const u32x4 Vr = rsrc_words(a.Vt + bkv * (vt_bytes / 2), vt_bytes);
  const int32_t* idx_row = FUSED ? a.idx + bkv * a.Lc : nullptr;
  const __amdgpu_buffer_rsrc_t Ir = __builtin_amdgcn_make_buffer_rsrc((void*)idx_row, 0, FUSED ? Lc * 4 : 0, 0x00020000);

  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, lo = lane & 31, hi = lane >> 5;
  const int rg = wave & 3, kg = wave >> 2;               // row group, key group
  const int koff = 32 * kg;                              // this wavefront's keys inside a 64-key tile
  const int q0 = qt * BMS;
  const int wrow0 = q0 + RW * rg;
  const int half_bit = (LISTS && a.block < BMS) ? 1 << ((RW * rg) / a.block) : 1;
  const float c = a.c;
  const float c_ = c;
  const float inv_c = 1.0f / c;

  // ---- fused form: zero rows of the full-length output between this workgroup's first selected token
  // and the next workgroup's, paced over the tile loop (see attend.hip)
  constexpr int LPR = D / 8, RPP = kThreads / LPR;
  const bool zfill = FUSED && a.Of != nullptr;
  const long long o_pitch16 = FUSED ? a.os.l / 8 : LPR;
  const int32_t* inv_row = nullptr;
  u32x4* zrow = nullptr;
  int z_hi = 0, zt = 0, zr = 0;
  int z_every = 1, z_count = 1;
  auto start_zero_rows = [&](int n_pipelined) {
    inv_row = a.inv + bkv * a.L;
    const int tok_lo = zero_bound(a.L, nq_tiles, qt);
    z_hi = zero_bound(a.L, nq_tiles, qt + 1);
    zrow = (u32x4*)(a.Of + a.os.head(b, h)) + (tid % LPR);
    zt = tok_lo + tid / LPR;
    zr = zt < z_hi ? inv_row[zt] : 0;
    z_every = max(1, (int)((float)n_pipelined / (float)max(1, (z_hi - tok_lo + RPP - 1) / RPP)));
  };
  auto zero_step = [&]() {
    if (zr < 0) __builtin_nontemporal_store(u32x4{0u, 0u, 0u, 0u}, zrow + (long long)zt * o_pitch16);
    zt += RPP;
    zr = zt < z_hi ? inv_row[zt] : 0;
  };

  // ---- key tiles, two per step
  TileGen gen;
  gen.plain = !LISTS;
  gen.plain_i = 0;
  gen.plain_n = (min(q0 + BMS, Lc) + BN - 1) / BN;
  gen.sub = gen.kb = gen.use = 0;
  gen.n_lists = 1;
  gen.block = BMS;
  gen.tiles_per_block = BMS / BN;
  gen.full = 1;
  int longest_list = 0;
#pragma unroll
  for (int j = 0; j < kMaxLists; ++j) { gen.list[j] = nullptr; gen.cnt[j] = gen.pos[j] = 0; gen.cur[j] = INT_MAX; }
  if (!gen.plain) {
    gen.block = a.block;
    gen.n_lists = a.block >= BMS ? 1 : BMS / a.block;    // row blocks of the list inside the 128 rows: 1 or 2
    gen.tiles_per_block = a.block / BN;
    gen.full = 0;
    const int nqb = (Lc + a.block - 1) / a.block;
    const int32_t* bl = a.block_list + bh * a.bl_head_stride;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
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
  auto next_step = [&]() -> Step {
    Step s;
    s.a = gen.next();
    s.b = s.a.k0 >= 0 ? gen.next() : Tile{-1, 0};
    return s;
  };

  // ---- staging: global memory -> LDS, two K tiles and two V tiles per step; tiles that do not exist are replaced by
  // tile 0 in the look-ups and loads: loaded, never used
  Stg stg;
  stg.init(smem, tid);
  int ktok[2][CH];
  auto row_off = [&](int tok) -> int { return FUSED ? (int)__umul24(tok, k_pitch) : tok * ROWB; };
  auto fetch_tok = [&](int (&tok)[CH], int k0) { stg.template look_up<FUSED>(Ir, max(k0, 0), tok); };
  auto load_k = [&](const int (&tok)[CH], int tile, int i) { stg.load_k(Kr, row_off(tok[i]), tile, tile + KHALF, i); };
  auto load_v = [&](int k0, int tile, int i) { stg.load_v(Vr, max(k0, 0), tile, i); };
  const int khalf = __builtin_amdgcn_readfirstlane(kg) * KHALF;   // this wavefront's keys: half kg of a K tile, 64 bytes of a V^T row

  f32x16 o[QS][ND];
  float m[QS], l[QS];
  m[0] = kNegBig;
  l[0] = 0.f;
#pragma unroll
  for (int dt = 0; dt < ND; ++dt) o[0][dt] = f32x16{0};

  // Ring roles at the top of the iteration of step j:
  //   K: kb0 = b_j, ka1 = a_(j+1), kb1 = b_(j+1) readable; kwa, kwb receive a_(j+2), b_(j+2) during the iteration
  //   V: va0 = a_j, vb0 = b_j readable; vwa, vwb receive a_(j+1), b_(j+1)
  int kb0 = 0, ka1 = KTILE, kb1 = 2 * KTILE, kwa = 3 * KTILE, kwb = 4 * KTILE;
  int va0 = NKT * KTILE, vb0 = va0 + VTILE, vwa = va0 + 2 * VTILE, vwb = va0 + 3 * VTILE;
  auto rotate = [&]() {
    const int r0 = kb0, r1 = ka1;
    kb0 = kb1; ka1 = kwa; kb1 = kwb; kwa = r0; kwb = r1;
    int t = va0; va0 = vwa; vwa = t;
    t = vb0; vb0 = vwb; vwb = t;
  };

  // ---- prologue: K of steps 0 and 1 and V of step 0 into LDS, S^T of the first half
  Step S0 = next_step(), S1 = next_step(), S2 = next_step();
  f32x16 sA[QS], sB[QS];
  uint32_t pA[QS][8], pB[QS][8];
  // half tile h of step S: first key and whether this wavefront takes part in it
  auto act = [&](const Tile& t) -> bool { return t.k0 >= 0 && (t.use & half_bit) && t.k0 + koff <= wrow0 + RW - 1; };
  bf16x8 qf[QS][NS];             // Q^T operand fragments of the wavefront's 32 rows (both key groups hold the same rows)
  {
    // Everything the first two steps need is requested in two rounds, first the look-ups, then the rows they name and V: two
    // memory latencies instead of six (with the merge below shared by both key groups: 901 of 3001
    // tokens x 32 heads 55.2 -> 54.1 us for the layer, 256 of 1024 x 4 32.3 -> 30.9).
    int qtok = wrow0 + lo, k0tok[2][CH], k1tok[2][CH];
    if (FUSED) qtok = __builtin_amdgcn_raw_buffer_load_b32(Ir, qtok * 4, 0, 0);
    fetch_tok(k0tok[0], S0.a.k0);
    fetch_tok(k0tok[1], S0.b.k0);
    fetch_tok(k1tok[0], S1.a.k0);
    fetch_tok(k1tok[1], S1.b.k0);
    fetch_tok(ktok[0], S2.a.k0);
    fetch_tok(ktok[1], S2.b.k0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < CH; ++i) load_k(k0tok[0], kwa, i);   // a_0 only serves the first S^T below; the slot is free again after the second barrier
    __builtin_amdgcn_sched_barrier(0);
    int qrow_off = qtok * ROWB;
    if (FUSED) qrow_off = wrow0 + lo < Lc ? (int)__umul24(qtok, q_pitch) : a.L * q_pitch;   // past the end: out of the buffer's range, reads zeros
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(Qr, qrow_off + 16 * hi + 32 * s, 0, 0);
      qf[0][s] = __builtin_bit_cast(bf16x8, v);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < CH; ++i) {
      load_k(k0tok[1], kb0, i);
      load_k(k1tok[0], ka1, i);
      load_k(k1tok[1], kb1, i);
      load_v(S0.a.k0, va0, i);
      load_v(S0.b.k0, vb0, i);
    }
    // (the zero rows' first look-ups while those are under way)
    if (zfill) start_zero_rows(gen.plain ? q0 / (2 * BN) - 1 : gen.tiles_per_block * longest_list / 2 - 3);
  }
  wait_loads();                                          // (the next wait is at the end of the first iteration, see attend.hip)
  lds_barrier();
  if (S0.a.k0 >= 0) stg.template qk<QS>(kwa + khalf, qf, sA);
  lds_barrier();
  if (act(S0.a)) {
    if (S0.a.k0 + koff + 31 > wrow0) mask_half<QS>(sA, S0.a.k0 + koff, hi, wrow0 + lo);
    softmax_max<ND, QS>(sA, c, m, l, o);
  }

  // ---- the pipelined iteration (all four tiles of this step and the next lie below the workgroup's first
  // row and are used by all its wavefronts): the chunk stream of attend.hip with this kernel's pointers
  constexpr int kPF = TSA_PF, kRing = TSA_RING, kChunks = 4 * NS;
  static_assert(NS == 8 || NS == 4, "chunk stream is laid out for d = 128 or 64");
  constexpr int CPB = kChunks / 4;
  static_assert(kChunks % kRing == 0 && kRing > kPF && kPF <= CPB, "fragment ring does not fit the chunk stream");
  bf16x8 kfr[kRing];
  // fragment fetch for chunk c: block 0 reads b of the current step (kb_), block 2 a of the next (ka_),
  // blocks 1 and 3 the V tiles a and b of the current step
  auto fetch = [&](int c, int kb_, int ka_, int va_, int vb_) {
    const int blk = c / CPB, i = c % CPB, slot = c % kRing;
    if (blk == 0) kfr[slot] = stg.k_frag(kb_ + khalf, i);
    else if (blk == 2) kfr[slot] = stg.k_frag(ka_ + khalf, i);
    else kfr[slot] = stg.v_frag((blk == 1 ? va_ : vb_) + 64 * kg, i / ND, i % ND);   // (64 bytes: two k-steps)
  };
  auto prime_ring = [&]() {
#pragma unroll
    for (int c = 0; c < kPF; ++c) fetch(c, kb0, ka1, va0, vb0);
  };
  // v_*: first keys of the V tiles of step 1; tok_*: first compacted rows of the K tiles of step 3
  auto fast_iter = [&](const int v_a, const int v_b, const int tok_a, const int tok_b) {
    float mxc[QS], mx[QS], ps0[QS], ps1[QS];
    f32x16 acc[QS];
#pragma unroll
    for (int c = 0; c < kChunks; ++c) {
      const int blk = c / CPB, i = c % CPB, slot = c % kRing;
      if (i == 0) {
        if (blk == 0 || blk == 2) __builtin_amdgcn_s_setprio(2);
        else __builtin_amdgcn_s_setprio(0);
      }
      // the first chunks of the next iteration read b of the next step: complete since the previous barrier
      if (c + kPF < kChunks) fetch(c + kPF, kb0, ka1, va0, vb0);
      else fetch(c + kPF - kChunks, kb1, kwa, vwa, vwb);
      // K of step 2 -> kwa, kwb; V of step 1 -> vwa, vwb; then the look-ups of step 3
      if (c < 2 * CH) load_k(ktok[c / CH], c < CH ? kwa : kwb, c % CH);
      else if (c < 4 * CH) load_v(c < 3 * CH ? v_a : v_b, c < 3 * CH ? vwa : vwb, c % CH);
      else if (c == 4 * CH) {
        fetch_tok(ktok[0], tok_a);
        fetch_tok(ktok[1], tok_b);
      }
      if (blk == 0 || blk == 2) {
        const f32x16 (&s_in)[QS] = blk == 0 ? sA : sB;
        uint32_t (&p_out)[QS][8] = blk == 0 ? pA : pB;
        constexpr int EPS = 16 / NS;
        if (i == 0) acc[0] = f32x16{0};
        acc[0] = mfma32(kfr[slot], qf[0][i], acc[0]);
#pragma unroll
        for (int e = 0; e < EPS; e += 2) {
          const int r = EPS * i + e;
          const float p0 = fast_exp2(s_in[0][r]);
          const float p1 = fast_exp2(s_in[0][r + 1]);
          if (r == 0) { ps0[0] = p0; ps1[0] = p1; }
          else { ps0[0] += p0; ps1[0] += p1; }
          p_out[0][r >> 1] = pack_bf16(p0, p1);
        }
        if (i == CPB - 1) {
          f32x16 (&s_out)[QS] = blk == 0 ? sB : sA;
          s_out[0] = acc[0];
          l[0] += ps0[0] + ps1[0];
        }
      } else {
        f32x16 (&s_in)[QS] = blk == 1 ? sB : sA;
        const uint32_t (&pb)[QS][8] = blk == 1 ? pA : pB;
        const int hf = i / ND, dt = i % ND;
        constexpr int EPC = 16 / CPB;
        const bf16x8 vf = kfr[slot];
        o[0][dt] = mfma32(vf, p_operand(pb[0], hf), o[0][dt]);
#pragma unroll
        for (int e = 0; e < EPC; ++e) s_in[0][EPC * i + e] = fmaf(s_in[0][EPC * i + e], c_, -m[0]);
        if (i == 0) mx[0] = s_in[0][0];
        if (EPC == 2) mx[0] = __builtin_fmaxf(__builtin_fmaxf(mx[0], s_in[0][2 * i]), s_in[0][2 * i + 1]);
        else {
#pragma unroll
          for (int e = 0; e < EPC; ++e) mx[0] = fmaxf(mx[0], s_in[0][EPC * i + e]);
        }
        if (i == CPB - 1) mxc[0] = fmaxf(mx[0], __shfl_xor(mx[0], 32));
      }
      __builtin_amdgcn_sched_barrier(0);
      if (c == 2 * CPB - 1) raise_max_rel<ND, QS>(mxc, m, l, o, sB);
    }
    wait_loads();
    if (FUSED && zfill && --z_count <= 0) {              // behind the wait, see attend.hip
      zero_step();
      z_count = z_every;
    }
    lds_barrier();
    raise_max_rel<ND, QS>(mxc, m, l, o, sA);
    rotate();
  };

  // ---- step loop
  auto tile_pipelined = [&](const Tile& t) -> bool { return t.k0 >= 0 && t.use == gen.full && t.k0 + BN <= q0; };
  auto pipelined = [&](const Step& s) -> bool { return tile_pipelined(s.a) && tile_pipelined(s.b); };
  while (S0.a.k0 >= 0) {
    if (pipelined(S0) && pipelined(S1)) {
#pragma unroll
      for (int r = 0; r < 16; ++r) sA[0][r] = fmaf(sA[0][r], c_, -m[0]);
      prime_ring();
      do {
        const Step S3 = next_step();
        fast_iter(S1.a.k0, S1.b.k0, S3.a.k0, S3.b.k0);
        S0 = S1; S1 = S2; S2 = S3;
      } while (pipelined(S0) && pipelined(S1));
      if (S0.a.k0 < 0) break;
#pragma unroll
      for (int r = 0; r < 16; ++r) sA[0][r] = (sA[0][r] + m[0]) * inv_c;
    }
    // general iteration: masks and per-wavefront decisions
    const Step S3 = next_step();
#pragma unroll
    for (int i = 0; i < CH; ++i) {
      if (S2.a.k0 >= 0) {
        load_k(ktok[0], kwa, i);
        load_k(ktok[1], kwb, i);
      }
      if (S1.a.k0 >= 0) {
        load_v(S1.a.k0, vwa, i);
        load_v(S1.b.k0, vwb, i);
      }
    }
    if (S3.a.k0 >= 0) {
      fetch_tok(ktok[0], S3.a.k0);
      fetch_tok(ktok[1], S3.b.k0);
    }
    if (act(S0.b)) stg.template qk<QS>(kb0 + khalf, qf, sB);   // (what the wavefront's rows see and nothing else, see attend.hip)
    if (act(S0.a)) {
      softmax_exp<QS>(sA, c, m, l, pA);
      stg.template pv<QS>(va0 + 64 * kg, 0, pA, o);
    }
    if (act(S0.b)) {
      if (S0.b.k0 + koff + 31 > wrow0) mask_half<QS>(sB, S0.b.k0 + koff, hi, wrow0 + lo);
      softmax_max<ND, QS>(sB, c, m, l, o);
      softmax_exp<QS>(sB, c, m, l, pB);
      stg.template pv<QS>(vb0 + 64 * kg, 0, pB, o);
    }
    if (act(S1.a)) {
      stg.template qk<QS>(ka1 + khalf, qf, sA);
      if (S1.a.k0 + koff + 31 > wrow0) mask_half<QS>(sA, S1.a.k0 + koff, hi, wrow0 + lo);
      softmax_max<ND, QS>(sA, c, m, l, o);
    }
    wait_loads();
    lds_barrier();
    S0 = S1; S1 = S2; S2 = S3;
    rotate();
  }

  // ---- fused form: the zero rows the loop did not get to
  auto flush_zero_rows = [&]() {
    // Latency-bound: a batch of look-ups is a memory round trip.  Sixteen rows per thread and batch, the
    // look-ups of the next batch requested before the stores of the current one (so that waiting for them
    // never includes waiting for those stores to be acknowledged).
    constexpr int kBatch = 16;
    if (zr < 0) __builtin_nontemporal_store(u32x4{0u, 0u, 0u, 0u}, zrow + (long long)zt * o_pitch16);
    int t0 = zt + RPP;
    int r[kBatch];
#pragma unroll
    for (int j = 0; j < kBatch; ++j) r[j] = t0 + j * RPP < z_hi ? inv_row[t0 + j * RPP] : 0;
    while (t0 < z_hi) {
      const int t1 = t0 + kBatch * RPP;
      int rn[kBatch];
#pragma unroll
      for (int j = 0; j < kBatch; ++j) rn[j] = t1 + j * RPP < z_hi ? inv_row[t1 + j * RPP] : 0;
#pragma unroll
      for (int j = 0; j < kBatch; ++j)
        if (r[j] < 0) __builtin_nontemporal_store(u32x4{0u, 0u, 0u, 0u}, zrow + (long long)(t0 + j * RPP) * o_pitch16);
#pragma unroll
      for (int j = 0; j < kBatch; ++j) r[j] = rn[j];
      t0 = t1;
    }
  };

  // ---- merge of the two key groups: each keeps half of the columns and hands the other half of its accumulators, with
  // (m, l), to its partner through LDS, so that both finish and store half of the rows' columns
  constexpr int NX = ND / 2;                             // d sub-tiles a wavefront keeps
  constexpr int NF = 2 + 16 * NX;                        // floats a lane hands over
  using Out = RowOut<D, NX, FUSED>;
  static_assert(8 * NF * 256 <= NKT * KTILE + NVT * VTILE && Out::kLds <= NF * 256, "the exchange does not fit the tile rings");
  Out out;
  out.look_up(idx_row, wrow0, Lc, lane);
  __syncthreads();                                       // every wavefront is done with the tiles
  float* give = (float*)smem + wave * (NF * 64) + lane;  // field f of this lane: give[f * 64]
  float* take = (float*)smem + (wave ^ 4) * (NF * 64) + lane;
  give[0] = m[0];
  give[64] = l[0];
#pragma unroll
  for (int dt = 0; dt < NX; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) give[(2 + 16 * dt + r) * 64] = kg ? o[0][dt][r] : o[0][NX + dt][r];
  __syncthreads();
  f32x16 ox[NX];
  float mn, lt;
  {
    const float mt = take[0], lx = take[64];
    mn = fmaxf(m[0], mt);
    const float a_own = fast_exp2(m[0] - mn), a_in = fast_exp2(mt - mn);
    // group 0's term is the fused one in both groups: the row sum and the columns do not depend on who adds
    lt = kg ? fmaf(lx, a_in, l[0] * a_own) : fmaf(l[0], a_own, lx * a_in);
#pragma unroll
    for (int dt = 0; dt < NX; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float own = kg ? o[0][NX + dt][r] : o[0][dt][r], in = take[(2 + 16 * dt + r) * 64];
        ox[dt][r] = kg ? fmaf(in, a_in, own * a_own) : fmaf(own, a_own, in * a_in);
      }
  }

  // ---- epilogue: normalise, round to bf16, store the rows (RowOut; the LDS that the partner's half came through, which
  // nobody else reads)
  lt += __shfl_xor(lt, 32);
  char* const lds_out = (char*)smem + (wave ^ 4) * (NF * 256);
  out.put(ox, lt > 0.f ? 1.0f / lt : 0.f, lds_out, lane);
  out.store(a, b, h, wrow0, Lc, 32 * NX * kg, lds_out, lane, [&]() { if (zfill) flush_zero_rows(); });
  if (a.lse && kg == 0 && hi == 0 && wrow0 + lo < Lc) a.lse[bh * a.Lc + wrow0 + lo] = (mn + log2f(lt)) * kLn2;
}

}  // namespace

hipError_t launch_attend_split(AttendArgs& a, int d, bool fused, hipStream_t st) {
  a.nq_tiles = (a.Lc + BMS - 1) / BMS;
  a.nk_tiles = (a.Lc + BN - 1) / BN;
  map_workgroups(a);
  const unsigned grid = grid_for(a);
  const auto go = [&](auto fused_tag, auto lists_tag) {
    constexpr bool F = decltype(fused_tag)::value, B = decltype(lists_tag)::value;
    if (d == 128) attend_split_kernel<128, F, B><<<grid, kThreadsS, 0, st>>>(a);
    else attend_split_kernel<64, F, B><<<grid, kThreadsS, 0, st>>>(a);
  };
  const std::true_type yes;
  const std::false_type no;
  if (fused) a.block_list ? go(yes, yes) : go(yes, no);
  else a.block_list ? go(no, yes) : go(no, no);
  return hipGetLastError();
}

}  // namespace tsa
