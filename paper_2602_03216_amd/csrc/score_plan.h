// How a scoring call is cut into workgroups: keys per workgroup and query heads that a workgroup serves at a time.  Plain host
// code, apart from the kernels so that it can be compiled and checked without a GPU.
#pragma once

namespace tsa {

constexpr int kScoreCUs = 256;
constexpr int kMinChunk = 256;               // keys per workgroup: at least this, a multiple of 128 (every tile size divides it)
// Up to that many chunk partials per query are folded at the start of pass 2 instead of in a launch of their own (5 us):
// 16 chunks cost pass 2 about 2 us (8K tokens x 32 KV heads: 4.7 + 15.8 -> 18.0 us for both), 49 to 64 chunks what the
// launch costs (12345 tokens x 8: 23.7 -> 24.3, 128K: 80.9 -> 82.1).
constexpr int kFoldChunks = 32;

// query sub-tiles; 4: two sets of two
inline int nqt_for(int last_q) { return last_q <= 32 ? 1 : (last_q <= 64 ? 2 : 4); }

// workgroups that the LDS tiles and the registers allow to be resident: two per CU with up to 64 queries, else one of twice
// the wavefronts
inline int resident_workgroups(int QP) { return QP <= 64 ? 2 * kScoreCUs : kScoreCUs; }

struct ScorePlan {
  int chunk, nchunks;          // keys per workgroup, workgroups per KV head
  int heads;                   // query heads per workgroup at a time: 4, 2 or 1
};

// As many heads per workgroup as the group has, up to `most`, unless the chunks leave CUs idle: then a workgroup takes fewer
// heads, and its wavefronts split the keys of every tile instead.  8 KV heads x 3001 tokens are 96 workgroups with four heads
// each: passes of 11.4 and 12.0 us; 192 with two: 9.8 and 9.8; 384 with one: 10.2 and 11.3, so half the CUs busy is where the
// line lies.
inline int heads_for(long long chunks, int g, int most) {
  int hpw = g >= 4 ? 4 : (g >= 2 ? 2 : 1);
  while (hpw > 1 && (hpw > most || chunks * ((g + hpw - 1) / hpw) <= kScoreCUs / 2)) hpw /= 2;
  return hpw;
}

// KVH: KV heads of all batch entries; g: query heads per KV head.
inline ScorePlan plan_score(int KVH, int g, int L, int d, int last_q) {
  // Keys per workgroup: long enough that the start-up of a workgroup (Q fragments, first K tile)
  // is amortised, short enough for as many workgroups as are resident, so the launch runs as a single round (65..128
  // queries, one per CU, 2 x 6001 tokens x 8 KV heads: 1.5 rounds of 256 keys 35.0 and 31.2 us, one round of 384 keys 24.8 and 22.3).
  long long c = (long long)L * KVH / resident_workgroups(32 * nqt_for(last_q));
  c = (c + 127) / 128 * 128;
  if (c < kMinChunk) c = kMinChunk;
  if (c > 8192) c = 8192;
  ScorePlan p;
  p.chunk = (int)c;
  p.nchunks = (L + p.chunk - 1) / p.chunk;
  p.heads = heads_for((long long)p.nchunks * KVH, g, 4);
  // Workgroups of two heads instead of four on chunks twice as long; where that leaves few enough chunks for pass 2 to fold,
  // the launch in between falls away, which is worth the second staging of every key as long as the passes
  // are short.  Whole scoring, 64 queries, four / two heads, us: 32 heads over 8 of K x 10007 tokens 33.4 / 30.3, 14000 34.7 / 32.2, 20000 (chunks of
  // 384 keys) 41.2 / 41.2, 32768 (512) 56.1 / 56.7, 131072 156 / 169; d = 64 x 16384 28.8 / 26.2; 28 over 4 x 12000 32.6 / 29.9; 40 over 8 x
  // 9001 47.9 / 32.0; 16 over 2 x 12000 23.7 / 21.4; 16 over 4 x 16000, d = 64, 17.3 / 17.6.  (One head on chunks four times as long: 28
  // over 4 x 30000 57 / 62.)  100 queries: 28 over 4 x 12000 59.7 / 52.9, 10 over 2 x 9000 31.1 / 23.6, 8 over 1 x 9000 25.1 / 22.7.
  // Not where a workgroup already takes one head, because longer chunks are then fewer workgroups: 4 over 1 x 8193 tokens, 64 queries,
  // 16.4 / 18.3, 100 20.6 / 23.0, 6 over 1 x 10000 16.5 / 18.0.  Nor for groups beyond 16 (32 over 1 x 9000 28.9 / 31.1).  Up to 32 queries, whose
  // passes are the staging, only for more than one workgroup of four heads per CU and groups below 8: 32 queries, 28 over 4 x 12000
  // 23.3 / 21.4, 32 over 8 x 10007 22.9 / 21.9, 40 over 8 x 9001 30.9 / 22.3; but 64 over 8 x 14000 35.8 / 38.7, and 16 queries, 16 over 4 x
  // 10000 15.3 / 16.2, 12 over 3 x 10000 13.1 / 14.9.
  const long long of_four = (long long)p.nchunks * KVH * ((g + 3) / 4);
  const bool pays = last_q > 32 ? p.heads >= 2 && g <= 16 : of_four > kScoreCUs && g < 8;
  if (g >= 4 && p.nchunks > kFoldChunks && p.nchunks <= 2 * kFoldChunks && p.chunk * d <= 384 * 128 && pays) {
    p.chunk *= 2;
    p.nchunks = (L + p.chunk - 1) / p.chunk;
    p.heads = heads_for((long long)p.nchunks * KVH, g, 2);
  }
  return p;
}

}  // namespace tsa
