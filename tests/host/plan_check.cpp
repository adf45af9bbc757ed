// CPU check of the library's sizing rules (plan.cpp; test code only). Built
// with g++ against the host-only stand-in of the HIP runtime header; one
// named check per run, exit status 0 and a last line "ok" on success.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <initializer_list>
#include <vector>

#include "../../paper_2606_18600_amd/csrc/kernels.hpp"

using namespace stage_k;

#define CHECK(c, ...)                                              \
  do {                                                             \
    if (!(c)) {                                                    \
      std::fprintf(stderr, "line %d: %s: ", __LINE__, #c);         \
      std::fprintf(stderr, __VA_ARGS__);                           \
      std::fprintf(stderr, "\n");                                  \
      std::exit(1);                                                \
    }                                                              \
  } while (0)

namespace {

int up(int a, int b) { return (a + b - 1) / b; }

// Key split of prefill attention: parts within the grid and the buffer, every
// part not empty and starting no later than its item's first position.
void prefill_parts_check() {
  int split = 0, whole = 0;
  for (int d : {64, 128})
    for (int n_kv : {1, 2, 8})
      for (int items : {1, 2, 5, 16, 61, 300})
        for (int longest : {1, 4, 9, 17, 40, 96, 400, 1000})
          for (size_t room : {(size_t)0, (size_t)1 << 16, (size_t)1 << 20, (size_t)1 << 26}) {
            float buf;
            const long long total = (long long)items * (longest + 1) / 2 + longest / 2;
            const PrefillParts p = prefill_split(items, n_kv, total, longest, d, &buf, room);
            if (p.stages == 0) {
              ++whole;
              CHECK(p.most == 1, "no split has one part");
              continue;
            }
            ++split;
            CHECK((size_t)items * n_kv * p.most * prefill_part_floats(d) <= room, "buffer");
            for (int nst = 1; nst <= longest; ++nst)
              for (int npos : {1, 16, 64, 128}) {
                const int p0 = nst * kPrefillStage - npos;  // an item of nst stages
                if (p0 < 0) continue;
                const int parts = prefill_parts(p.stages, p0, nst);
                CHECK(parts >= 1 && parts <= p.most, "%d of %d parts", parts, p.most);
                CHECK((parts - 1) * p.stages < nst, "empty part");
                CHECK((parts - 1) * p.stages * kPrefillStage <= p0, "part past position %d", p0);
              }
          }
  CHECK(split > 100 && whole > 100, "%d split, %d whole", split, whole);
  // few chunks behind long prefixes are split, many or short ones are not
  float buf;
  const size_t room = (size_t)1 << 26;
  CHECK(prefill_split(1, 1, 64, 64, 128, &buf, room).most > 1, "one position behind 4000 keys");
  CHECK(prefill_split(4, 2, 4 * 95, 95, 128, &buf, room).most > 1, "64 behind 6000, two kv heads");
  CHECK(prefill_split(12, 8, 12 * 58, 58, 128, &buf, room).most > 1, "191 behind 3535, 8 heads");
  CHECK(prefill_split(128, 8, 128 * 960, 960, 128, &buf, room).stages == 0, "2048 behind 61440");
  CHECK(prefill_split(25, 8, 25 * 4, 7, 128, &buf, room).stages == 0, "400 rows of one prompt");
}

// Products of at most 32 rows: the planned K ranges are what the launcher
// takes (every range not empty), never more than the plan they replace, and
// the stream kernel is chosen at the shapes made for it.
void stream_check() {
  int taken = 0;
  for (int N = 64; N <= 65536; N += N < 4096 ? 64 : 1088)
    for (int K = 64; K <= 28672; K += K < 1024 ? 64 : 896)
      for (int most : {1, 2, 5, 8, 32}) {
        if (N % 64 || K % 64) continue;
        const int s = stream_splits(N, K, most, false);
        if (s == 0) continue;
        ++taken;
        CHECK(s >= 1 && s <= most, "N %d K %d: %d of %d ranges", N, K, s, most);
        const int kb = skinny_kp_used(K, s, false) ? skinny_kp_kb_len(K, s) : skinny_kb_len(K, s);
        CHECK(up(K, kb) == s, "N %d K %d: %d ranges of %d", N, K, s, kb);
        for (int M : {1, 16, 17, 32}) {
          const int f = stream_fragments(M, N, K, s, false);
          CHECK(f == 2 || f == 4, "N %d K %d M %d", N, K, M);
          CHECK(N / 64 * s * (f == 2 ? 2 : 1) <= kStreamBlocks, "blocks");
        }
      }
  CHECK(taken > 1000, "%d plans", taken);
  for (int N : {1280, 512, 1408}) CHECK(stream_fragments(32, N, 704, 1, false) == 2, "N %d", N);
  CHECK(stream_splits(8192, 512, 8, false) == 2, "two K ranges of 256");
  CHECK(stream_fragments(1, 8192, 512, 2, false) == 4, "whole groups");
  CHECK(stream_fragments(32, 8320, 256, 1, true) == 4, "SwiGLU of 130 groups");
  CHECK(stream_fragments(16, 16512, 384, 1, true) == 4, "SwiGLU of 258 groups, 16 rows");
  CHECK(stream_fragments(17, 16512, 384, 1, true) == 0, "SwiGLU of 258 groups, 17 rows");
  CHECK(stream_fragments(33, 512, 256, 1, false) == 0, "33 rows");
}

TiledShape shape(int H, int nq, int nkv, int d, int F) {
  TiledShape t;
  t.hidden = H;
  t.qw = nq * d;
  t.qkvw = (nq + 2 * nkv) * d;
  t.ffn = F;
  t.max_tokens = 2176;
  t.tail_rows = 128;
  t.gate_up_room = mid_capacity(t.max_tokens, t.qkvw);
  return t;
}

// Products whose tiles fill exactly half of the CUs are split for a long K
// only; fewer tiles split whatever K is.
void half_round_check() {
  const TiledShape t = shape(8192, 64, 8, 128, 28672);
  struct { int T, N; } half[] = {{769, 8192}, {1024, 8192}, {1793, 4096}, {2048, 4096}, {200, 32768}};
  for (auto h : half) {
    for (int K : {512, 1024, 2048}) CHECK(mid_splits(t, h.T, h.N, K) == 0, "%d x %d K %d", h.T, h.N, K);
    if (h.N <= 8192)
      for (int K : {3584, 4096, 8192, 28672})
        CHECK(mid_splits(t, h.T, h.N, K) == 2, "%d x %d K %d", h.T, h.N, K);
  }
  CHECK(mid_splits(t, 768, 8192, 1024) == 2, "96 tiles");
  CHECK(mid_splits(t, 256, 8192, 1024) == 8, "32 tiles");
  CHECK(mid_splits(t, 1025, 8192, 28672) == 0, "160 tiles");
}

// Rows past the last whole row of tiles: a step whose whole tiles fill exactly
// half of the CUs (or more) in O and down keeps its tail, one whose whole tiles
// fill less is split over K instead.
void row_tail_check() {
  struct { TiledShape t; int T, rows; bool qkv; } cases[] = {
      {shape(8192, 64, 32, 128, 22016), 1025, 1, true},   // QKV: 256 tiles of 1024 rows
      {shape(8192, 64, 32, 128, 22016), 1152, 128, true},
      {shape(8192, 64, 32, 128, 22016), 1153, 0, false},  // more rows than the skinny kernels take
      {shape(4096, 32, 16, 128, 14336), 2049, 1, true},
      {shape(4096, 32, 16, 128, 14336), 2176, 128, true},
      {shape(8192, 64, 8, 128, 28672), 1100, 76, false},
      {shape(8192, 64, 8, 128, 28672), 2176, 128, false},  // 320 or 360 tiles: two rounds either way
      {shape(8192, 64, 8, 128, 28672), 800, 0, false},    // O, down: 96 tiles of 768 rows
      {shape(8192, 64, 8, 128, 28672), 200, 0, false},    // no whole row of tiles
      {shape(8192, 64, 8, 128, 28672), 2048, 0, false},
  };
  for (auto& c : cases) {
    const int rt = row_tail(c.t, c.T);
    CHECK(rt == c.rows, "H %d T %d: %d rows", c.t.hidden, c.T, rt);
    CHECK(row_tail_for(c.t, c.T, rt, c.t.qkvw) == c.qkv, "H %d T %d", c.t.hidden, c.T);
  }
}

// Gate-up products of small steps: split over K where that is faster than one
// range on 128 x 128 tiles, not where the planes and the second pass cost more
// than they save (a short K, tiles that fill the CUs).
void gate_up_check() {
  auto splits = [](int T, int F, int K) { return gate_up_splits(shape(K, 64, 16, 128, F), T); };
  struct { int T, N, K; } whole[] = {
      {768, 2048, 1024}, {256, 1024, 1024}, {432, 3584, 1024}, {200, 7168, 1024}, {512, 7168, 2048},
      {256, 14336, 2048}, {192, 16384, 2048}, {400, 2048, 512}, {1536, 2048, 2048}, {1300, 3584, 3072},
  };
  for (auto c : whole) CHECK(splits(c.T, c.N / 2, c.K) == 0, "%d x %d K %d", c.T, c.N, c.K);
  struct { int T, N, K, sp; } split[] = {
      {150, 7168, 8192, 8}, {600, 7168, 8192, 2}, {400, 14336, 8192, 2}, {150, 14336, 8192, 4},
      {200, 3584, 4096, 8}, {513, 512, 2048, 8},
      {130, 7168, 2048, 8}, {160, 11264, 2560, 4}, {130, 14336, 2560, 4}, {160, 24576, 2048, 2},
  };
  for (auto c : split) {
    const int sp = splits(c.T, c.N / 2, c.K);
    CHECK(sp == c.sp, "%d x %d K %d: %d", c.T, c.N, c.K, sp);
  }
  for (int T = 129; T <= 2176; T += 61)
    for (int F = 128; F <= 28672; F += 896)
      for (int K = 512; K <= 8192; K *= 2) {
        TiledShape t = shape(K, 64, 16, 128, F);
        t.gate_up_room = (size_t)1 << 22;
        const int sp = gate_up_splits(t, T);
        CHECK(sp == 0 || sp == 2 || sp == 4 || sp == 8, "%d", sp);
        if (sp == 0) continue;
        CHECK(2 * F % 256 == 0 && K % (64 * sp) == 0, "tiles");
        CHECK((size_t)sp * T * 2 * F <= t.gate_up_room, "room");
        CHECK(up(T, 256) * (2 * F / 256) * sp <= t.cus, "one round");
      }
}

// 129-176 rows of SwiGLU past the last row of tiles: on the skinny kernel
// where its pass is cheaper than the partial round it saves.
void swiglu_tail_check() {
  // rounds of 256-row tiles that the other tilings need less those that the
  // whole rows of tiles need: 0.7 (two rounds of 192-row tiles), 0.9, 1
  for (int K : {1024, 2048, 5120, 8192}) {
    CHECK(swiglu_tail_rounds(166, 16384, K) > 0.7, "narrow, K %d", K);
    CHECK(swiglu_tail_rounds(129, 34816, K) > 0.7, "K %d", K);
    CHECK(swiglu_tail_rounds(176, 40960, K) < 0.9, "K %d", K);
    CHECK(swiglu_tail_rounds(129, 57344, K) < 1 && swiglu_tail_rounds(144, 51200, K) < 1, "K %d", K);
  }
  CHECK(swiglu_tail_rounds(176, 57344, 1024) > 1 && swiglu_tail_rounds(176, 57344, 8192) < 1, "K");
  CHECK(swiglu_tail_rounds(128, 57344, 8192) == 57344 / 78000.0, "up to 128 rows");
}

// 129-192 rows split over K: the skinny kernel for long K ranges, and for
// short ranges and past 176 rows where the launch fills most CUs.
void rows192_check() {
  for (int k : {64, 128, 256, 448, 512, 768, 896}) {
    for (int M : {129, 160, 176, 192}) {
      for (int blocks : {112, 128, 160}) CHECK(!rows192_skinny(M, blocks, k), "%d rows, %d", M, k);
      for (int blocks : {8, 64, 96})
        CHECK(rows192_skinny(M, blocks, k) == (k >= 640 && M <= 160), "%d rows, %d", M, k);
    }
    for (int M : {129, 144, 160, 176})
      CHECK(rows192_skinny(M, 192, k) && rows192_skinny(M, 256, k), "%d rows, %d", M, k);
    CHECK(!rows192_skinny(190, 192, k) && !rows192_skinny(190, 224, k), "190 rows, %d", k);
    CHECK(rows192_skinny(190, 256, k), "190 rows of 256 blocks, %d", k);
  }
  for (int k : {1024, 2048, 3584, 8192}) {
    for (int blocks : {8, 64, 128, 256})
      for (int M : {129, 144, 160, 176}) CHECK(rows192_skinny(M, blocks, k), "%d rows, %d", M, k);
    CHECK(rows192_skinny(191, 256, k) && rows192_skinny(177, 224, k), "most CUs");
    CHECK(!rows192_skinny(191, 128, k) && !rows192_skinny(177, 64, k), "few CUs");
    CHECK(!rows192_skinny(128, 256, k) && !rows192_skinny(193, 256, k), "rows");
  }
}

// Key splits of decode sequences: 32 each unless few long sequences gain by
// more; never more for tokens whose merge would cost more than it saves.
void decode_splits_check() {
  auto most = [](std::initializer_list<int> ctx, int n_kv, int group, int j = 0) {
    const DecodeSplits s = decode_splits(ctx.begin(), (int)ctx.size(), n_kv, group, 256);
    return s.most((ctx.begin()[j] + kBlock) / kBlock);
  };
  for (int kv : {1, 2, 4}) {
    CHECK(most({40000}, kv, 16) <= 64 && most({60000}, kv, 16) <= 64, "kv %d, 16 heads", kv);
    CHECK(most({10000}, kv, 16) == 32, "kv %d, 16 heads, 10000 keys", kv);
    CHECK(most({40000}, kv, 8) == 64 && most({10000}, kv, 8) == 48, "kv %d", kv);
    CHECK(most({1000}, kv, 8) == 32, "kv %d, 1000 keys", kv);
  }
  CHECK(most({40000, 40000, 40000}, 8, 8) == 32, "24 pairs");
  CHECK(most({60000, 20000, 40000}, 8, 8) == 47 && most({60000, 20000, 40000}, 8, 8, 1) == 32,
        "24 uneven pairs");
  CHECK(most({40000, 20000, 40000, 40000}, 8, 8) == 32, "a block per CU already");
  CHECK(most({10000, 10000, 10000, 10000, 10000, 10000, 10000, 10000, 10000, 10000}, 1, 16) == 32,
        "10 pairs of 16 heads");
  CHECK(most({60000, 60000, 60000, 60000, 60000}, 8, 8) > 1000, "40 pairs: as the waves need");
  for (int nd : {1, 3, 7, 64, 200}) {  // any step: a positive count for every sequence
    std::vector<int32_t> ctx(nd);
    for (int j = 0; j < nd; ++j) ctx[j] = j * 7919 % 65000;
    for (int kv : {1, 3, 8, 32})
      for (int g : {1, 16}) {
        const DecodeSplits s = decode_splits(ctx.data(), nd, kv, g, 256);
        for (int c : ctx) CHECK(s.most((c + kBlock) / kBlock) >= kMaxSplits, "nd %d", nd);
      }
  }
  CHECK(decode_splits(nullptr, 0, 8, 8, 256).most(1) == kMaxSplits, "no sequence");
}

}  // namespace

int main(int argc, char** argv) {
  const char* name = argc > 1 ? argv[1] : "";
  if (!std::strcmp(name, "prefill_parts"))
    prefill_parts_check();
  else if (!std::strcmp(name, "stream"))
    stream_check();
  else if (!std::strcmp(name, "half_round"))
    half_round_check();
  else if (!std::strcmp(name, "row_tail"))
    row_tail_check();
  else if (!std::strcmp(name, "gate_up"))
    gate_up_check();
  else if (!std::strcmp(name, "swiglu_tail"))
    swiglu_tail_check();
  else if (!std::strcmp(name, "rows192"))
    rows192_check();
  else if (!std::strcmp(name, "decode_splits"))
    decode_splits_check();
  else
    return 2;
  std::puts("ok");
  return 0;
}
