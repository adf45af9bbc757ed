// Host-side sizing rules shared by the launchers and the stage runtime: the K
// ranges of decode products and the kernel of those of at most 32 rows, the K
// ranges of small tiled steps and the last rows of large ones, and the
// positions of a prefill attention work item and the split of its keys. Plain
// host code (no HIP calls).
#include <algorithm>
#include <cstdlib>

#include "kernels.hpp"

namespace stage_k {

int skinny_kb_len(int K, int splits) {
  int kb = (K + splits - 1) / splits;
  return (kb + 63) / 64 * 64;
}

int skinny_splits(int N, int K, int target_blocks, int max_splits) {
  const int col_blocks = (N / 64 + kSkinnyWaves - 1) / kSkinnyWaves;
  int s = std::max(1, target_blocks / col_blocks);
  s = std::min(s, std::min(max_splits, K / 64));
  // the number of K ranges actually launched after rounding the range up
  const int kb = skinny_kb_len(K, s);
  return (K + kb - 1) / kb;
}

bool skinny_kp_enabled() {
  static const bool on = [] {
    const char* v = std::getenv("STAGE_SKINNY_KP");
    return !(v && *v && std::atoi(v) == 0);
  }();
  return on;
}

bool skinny_kp_used(int K, int splits, bool swiglu) {
  return !swiglu && splits > 1 && K % 128 == 0 && skinny_kp_enabled();
}

int skinny_kp_kb_len(int K, int splits) {
  int kb = (K + splits - 1) / splits;
  return (kb + 127) / 128 * 128;
}

int skinny_kp_splits(int N, int K, int target_blocks, int max_splits) {
  const int col_blocks = (N / 64 + kSkinnyKpGroups - 1) / kSkinnyKpGroups;
  int s = std::max(1, target_blocks / col_blocks);
  s = std::min(s, std::min(max_splits, K / 128));
  const int kb = skinny_kp_kb_len(K, s);
  return (K + kb - 1) / kb;
}

int stream_fragments(int M, int N, int K, int splits, bool swiglu) {
  if (M > kStreamRows) return 0;
  const int groups = N / 64;
  if (2 * groups * splits <= kStreamBlocks) return 2;
  if (swiglu && M <= 16 && groups <= 2 * kStreamBlocks) return 4;
  if (groups * splits > kStreamBlocks) return 0;
  return swiglu || K / splits <= kStreamMaxRange ? 4 : 0;
}

int stream_splits(int N, int K, int max_splits, bool swiglu) {
  const int groups = N / 64;
  if (groups > kStreamBlocks) return 0;
  const int per = groups <= 64 ? 2 : 1;  // blocks per group and K range
  int s = 1;
  if (!swiglu) {
    s = std::max(1, std::min({kStreamBlocks / (per * groups), max_splits, K / 256}));
    // the K ranges the launcher will take (gemm_skinny)
    const int kb = skinny_kp_used(K, s, false) ? skinny_kp_kb_len(K, s) : skinny_kb_len(K, s);
    s = (K + kb - 1) / kb;
  }
  const int frags = stream_fragments(1, N, K, s, swiglu);
  const int blocks = groups * s * (frags == 2 ? 2 : 1);
  return frags && (blocks * 10 >= kStreamBlocks * 7 || K <= 2048) ? s : 0;
}

PrefillParts prefill_split(int n_items, int n_kv, long long total, int longest, int head_dim,
                           float* buf, size_t room) {
  // Two blocks per CU (at the 70B shape: 154 rows behind 3535 keys 83 us on
  // 80 blocks, 51 + 6 for the combining pass on 256, 38 + 8 on 512, 42 + 11
  // on 768; 256 rows behind 30000 keys 600, 361 + 6, 283 + 9, 304 + 10; 512
  // rows behind 8000 keys 202, 198, 161 + 10, 167 + 11), parts of at least 4
  // stages, and only where that pays: a stage takes about 1.3 us with a block
  // per CU and 2.4 with two, the combining pass 10 (400 rows behind 1000 keys
  // gain nothing; 150 rows and one kv head behind 700, 10 stages' chain less
  // on a nearly empty chip, 14 us per layer). At head_dim 64 as well: of 110
  // random steps of 1-16 heads per group and 150-6000 cached keys none is
  // slower than unsplit beyond noise, those of 500 keys and more 4-40% faster.
  constexpr int kBlocks = 2 * kCus, kMinStages = 4;
  const long long blocks = (long long)n_items * n_kv;
  if (blocks >= kBlocks) return PrefillParts{};
  long long stages = std::max<long long>(kMinStages, (total * n_kv + kBlocks - 1) / kBlocks);
  for (; longest > stages; stages *= 2) {
    const long long most = (longest + stages - 1) / stages;
    const bool pays = blocks * most <= kBlocks / 2 ? longest - stages >= 8
                                                   : 13LL * longest > 24 * stages + 100;
    if (!pays) break;
    if ((size_t)(blocks * most) * prefill_part_floats(head_dim) <= room)
      return PrefillParts{buf, (int32_t)stages, (int32_t)most};
  }
  return PrefillParts{};
}

// More splits shorten a long sequence's chain of keys but lengthen its merge,
// one block per (token, kv head) that reads every split (kv1 x 16 heads, one
// token of 60000 keys, us per layer: 32 splits 91, 64 72, 400 137; x 8 heads 82,
// 60, 63). So with up to 12 (token, kv head) pairs sequences of ~14000 keys and
// more get 64 each, of ~6400 48 (16 heads per group: 48 from 14000 on, up to 6
// pairs); from 33 pairs on, where 32 splits each are 1.25 blocks per CU and
// more, whatever evens out the waves (5 sequences of 60000 keys, 8 kv heads:
// 246 -> 220). In between, 32 each; a longer sequence in proportion, if a block
// per CU still holds them all (3 sequences of 18000-60000 keys, 8 kv heads: 127
// -> 115; but 4 of 20000-40000, 256 blocks: 125 -> 153).
DecodeSplits decode_splits(const int32_t* ctx_lens, int nd, int n_kv, int group, int cus) {
  constexpr int kUnlimited = 1 << 20;
  DecodeSplits r;
  if (nd <= 0) return r;
  long long total = 0;
  for (int j = 0; j < nd; ++j) total += (ctx_lens[j] + kBlock) / kBlock;
  r.mean = std::max(1LL, total / nd);
  const long long pairs = (long long)nd * n_kv;
  const bool wide = group > 8;
  if (pairs <= (wide ? 6 : 12) && r.mean >= 900) {
    r.base = wide ? 48 : 64;
  } else if (pairs <= 8 && r.mean >= 400 && !wide) {
    r.base = 48;
  } else if (pairs > 32) {
    r.even = true;
    if (r.mean >= 500 && !wide) r.base = kUnlimited;
  } else {
    long long items = 0;
    for (int j = 0; j < nd; ++j) items += r.most((ctx_lens[j] + kBlock) / kBlock);
    r.even = items * ((n_kv + 3) / 4) > cus || (wide && r.mean < 900);
  }
  return r;
}

// Product and consumer on 192-row tiles -> skinny, at 129 / 176 / 190 rows:
// [2048, 3584] in 8 ranges 20 -> 20 / 21 -> 23 / 22 -> 24 us; [8192, 8192] in 8
// (256 blocks) 45 -> 41 / 48 -> 45 / 50 -> 47; [2048, 8192] in 8 (64 blocks) 28
// -> 27 / 30 -> 30 / 30 -> 32. 12 row tiles leave the skinny waves no registers
// to read ahead, which shows once a launch is not bound by HBM. Ranges below
// 1024 are over before their reads ahead pay for their final sums, but with
// most CUs at work the kernels around a tiled product lose more (two norms, RoPE
// and attention 2-3 us in all): whole layers of O and down in 8 ranges, tiles
// -> skinny at 130 / 160 / 190 rows, N = 4096 (128 blocks) and ranges of 768
// 108 -> 114 / 112 -> 118 / 119 -> 128 us, 5120 122 -> 125 / 128 -> 131 / 138 ->
// 143, 6144 136 -> 134 / 143 -> 143 / 154 -> 156, 7168 151 -> 146 / 160 -> 157 /
// 170 -> 171, 8192 164 -> 159 / 174 -> 170 / 186 -> 186 (one rank of 4, ranges
// of 896, 8192: 177 -> 172 / 187 -> 182 / 200 -> 197). With few blocks the
// final sums are short, and ranges from 640 on pay for them up to 160 rows (32
// to 96 blocks, ranges of 768, product alone at 129 / 160 / 176 / 190 rows 18.3
// -> 17.3 / 18.7 -> 18.4 / 19.0 -> 19.3 / 19.4 -> 21.2).
bool rows192_skinny(int M, long blocks, int k_len) {
  if (M <= 128 || M > 192) return false;
  if (k_len < 1024)
    return 8 * blocks > (M <= 176 ? 5 : 7) * kCus ||
           (k_len >= 640 && M <= 160 && 8 * blocks <= 3 * kCus);
  return M <= 176 || blocks > 128;
}

size_t mid_capacity(int max_tokens, int N) {
  return std::max((size_t)kMidRows * N,
                  std::min(kMidElems, (size_t)kMaxMidSplits * max_tokens * N));
}

// At exactly half of the CUs 128 x 128 tiles would fill their two slots per
// CU, and what two ranges save grows with K while their planes cost the same
// (product and RMSNorm, one range -> two, at 900 x 8192 / 1800 x 4096: K =
// 1024 45 -> 50 / 37 -> 51 us, 2048 63 -> 61 / 54 -> 62, 3584 90 -> 76 / 79 ->
// 78, 8192 162 -> 125 / 151 -> 126, 28672 528 -> 361 / 514 -> 364): split from
// kHalfRoundK on.
int mid_splits(const TiledShape& t, int T, int N, int K) {
  constexpr int kHalfRoundK = 3072;
  if (N % 256 != 0) return 0;
  const int tiles = (T + 255) / 256 * (N / 256);
  if (2 * tiles > t.cus || (2 * tiles == t.cus && K < kHalfRoundK)) return 0;
  int best = 0;
  for (int sp = 2; sp <= kMaxMidSplits; sp *= 2)
    if (tiles * sp <= t.cus && K % (64 * sp) == 0 &&
        (size_t)sp * T * N <= mid_capacity(t.max_tokens, N))
      best = sp;
  return best;
}

// Times in us, fitted to 846 products of 129-2048 rows, N = 1024-32768 and K =
// 512-8192 (within 10%, a few within 25%). Unsplit: one range of K on 128 x
// 128 tiles, one per CU or two. Split: a range on 256-row tiles, the planes
// written and read, two launches' ends; for 192 rows and fewer fitted to what
// 264 whole layers take with each number of ranges, since there the kernels
// around the product gain as well. What saves less than 7% is left unsplit.
// Layers are 0.1 us from their best choice on average up to 192 rows (3 at
// most), 0.3 of 245 layers of 224-900 rows (7). (2 F = 7168: 150 rows, K = 8192
// 87 -> 36 us, but 432 rows, K = 1024 16 -> 25; 2 F = 14336, 130 rows, K =
// 2560: layer of 101 us unsplit, 98 in 2 ranges, 93 in 4.)
int gate_up_splits(const TiledShape& t, int T) {
  const int N = 2 * t.ffn, K = t.hidden;
  if (N % 256 != 0) return 0;
  const long tiles = (long)(T + 255) / 256 * (N / 256);
  const long tiles128 = (long)(T + 127) / 128 * (N / 128);
  // (just past one per CU most of them still have a CU to themselves)
  const double unsplit = tiles128 <= t.cus           ? 5 + K / 96.0
                         : 4 * tiles128 <= 5 * t.cus ? 6 + K / 70.0
                         : 2 * tiles128 <= 3 * t.cus ? 6 + K / 62.0
                                                     : 6 + K / 57.0;
  int best = 0;
  double cost = 0.93 * unsplit;
  for (int sp = 2; sp <= kMaxMidSplits; sp *= 2) {
    if (tiles * sp > t.cus || K % (64 * sp) != 0 || (size_t)sp * T * N > t.gate_up_room) break;
    const double range = (double)K / sp, plane = 1e-6 * sp * T * N;
    const double c = T <= 192 ? 12 + range / 76 + 0.7 * plane : 10 + range / 58 + 1.2 * plane;
    if (c < cost) best = sp, cost = c;
  }
  return best;
}

double swiglu_tail_rounds(int rows, int N, int K) {
  if (rows <= 128) return N / 78000.0;  // the weights at ~6.3 TB/s, a tile at ~5.3 TFLOP/s
  // An eighth more at 144 rows and growing with the rows; fewer than ~190
  // blocks of 256 columns no longer keep HBM busy, and the launch is one more
  // (166 rows past 1024 at N = 16384, K = 2048: 76 us on two rounds of 192-row
  // tiles, 91 so; 176 past 256 at 40960, 1024: 52 and 60; but past 512 at
  // 40960, 8192 662 and 522).
  const double pass = N / 68000.0 * (1 + (rows - 144) / 256.0);
  return std::max(0.72, pass) + 100.0 / K;
}

int row_tail(const TiledShape& t, int T) {
  const int rt = T % 256, T0 = T - rt;
  if (rt == 0 || rt > t.tail_rows || T0 < 256) return 0;
  // (exactly half of the CUs at T0 are more than half at T: nothing is split
  // there. One layer of 1100 rows with 64 column tiles of QKV: 1664 us with
  // the tail, 1700 without.)
  auto split = [&](int N, int K) {
    return 2 * (T0 / 256 * (N / 256)) < t.cus && mid_splits(t, T0, N, K) > 0;
  };
  if (split(t.qkvw, t.hidden) || split(t.hidden, t.qw) || split(t.hidden, t.ffn)) return 0;
  return rt;
}

bool row_tail_for(const TiledShape& t, int T, int rt, int N) {
  if (rt == 0 || N % 256 != 0) return false;
  const long cols = N / 256;
  const long with = (T + 255) / 256 * cols, without = (T - rt) / 256 * cols;
  return (with + t.cus - 1) / t.cus > (without + t.cus - 1) / t.cus;
}

int prefill_item_positions(DType dt, int group) {
  (void)dt;
  return kPrefillRows / group;
}

}  // namespace stage_k
