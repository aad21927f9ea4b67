// The host rules that choose the grid of a decode launch (file-local in csrc/decode_kernels.hip, hence the include): over all
// numbers of pairs, records and fp16 rows, and over batches of different lengths.  No kernel is launched.
#include <cstdio>
#include <random>
#include "decode_kernels.hip"

#define CHECK(cond, ...)                                                           \
  do {                                                                             \
    if (!(cond)) {                                                                 \
      fprintf(stderr, "%s:%d: check failed: %s: ", __FILE__, __LINE__, #cond);     \
      fprintf(stderr, __VA_ARGS__);                                                \
      fprintf(stderr, "\n");                                                       \
      exit(1);                                                                     \
    }                                                                              \
  } while (0)

using namespace mixkvq;

static CacheView view_of(int B, int Hkv, int g) {
  CacheView v{};
  v.cfg.B = B; v.cfg.Hkv = Hkv; v.cfg.Hq = Hkv * g;
  v.P = B * Hkv;
  v.g = g;
  return v;
}

static int chain_of(int units, const DecodeGrid& d) { return (units + d.n_waves * d.n_splits - 1) / (d.n_waves * d.n_splits); }

static void equal_lengths(int P, int g, int n_blocks, int n_fp16) {
  const CacheView v = view_of(P, 1, g);
  const int subs = (n_fp16 + 31) / 32, units = n_blocks + subs, cap = max_splits_for(P);
  int ns4, ns8;
  DecodeGrid four, got;
  choose_splits(v, n_blocks, n_fp16, false, &ns4, &four);
  choose_splits(v, n_blocks, n_fp16, true, &ns8, &got);
#define AT "P %d, %d heads, %d records, %d fp16 rows: %d workgroups of %d (%d of four, ceiling %d)", P, g, n_blocks, n_fp16, got.n_splits, got.n_waves, four.n_splits, cap
  CHECK(ns4 == ns8 && ns4 >= 1 && ns4 <= cap, AT);
  CHECK(four.n_waves == 4 && (got.n_waves == 4 || got.n_waves == 8), AT);
  CHECK(got.n_waves == 8 ? got.n_splits <= four.n_splits : got.n_splits == four.n_splits, AT);
  // what launch_decode asks before it takes the matrix-core kernel
  CHECK(got.n_splits >= 1 && (got.n_splits <= cap || four.n_splits > cap), AT);
  CHECK(got.n_splits * got.n_waves >= subs, AT);                                            // a sub-unit per wavefront at most
  CHECK(got.n_splits == 1 || (got.n_splits - 1) * got.n_waves < units, AT);                 // every workgroup has a unit
  CHECK(chain_of(units, got) <= chain_of(units, four) || four.n_splits > cap, AT);
  // workgroups of eight in one round, or one a pair
  CHECK(got.n_waves == 4 || P * got.n_splits <= 256 || got.n_splits == 1 || four.n_splits > cap, AT);
  if (got.n_splits <= cap)      // the partials it writes are those the size was given for
    CHECK((size_t)P * got.n_splits * v.g * kPartStride * sizeof(float) <= decode_launch_partials_bytes(v, n_blocks, n_fp16), AT);
#undef AT
}

// pairs, heads of a pair, records, fp16 rows: the grid that the timings beside eight_wavefronts speak for
static const struct { int P, g, n_blocks, n_fp16, n_splits, n_waves; } kLines[] = {
    {24, 7, 70, 41, 9, 8},    {32, 7, 256, 37, 8, 8},   {32, 1, 62, 37, 8, 8},    {28, 7, 128, 37, 9, 8},  {188, 4, 7, 94, 1, 8},
    {36, 6, 128, 37, 14, 4},  {36, 7, 128, 37, 7, 8},   {34, 1, 500, 37, 15, 4},  {34, 8, 328, 37, 7, 8},  {40, 8, 62, 37, 12, 4},
    {40, 7, 256, 37, 12, 4},  {112, 1, 26, 125, 4, 4},  {3, 2, 239, 59, 31, 8},   {1, 6, 126, 32, 32, 4},  {1, 7, 126, 32, 16, 8},
    {1, 7, 94, 32, 24, 4},    {1, 7, 98, 32, 13, 8},    {1, 1, 130, 32, 17, 8},   {14, 7, 56, 50, 15, 4},  {1, 1, 32, 3, 9, 4},
    // more than one round of workgroups of eight
    {146, 7, 200, 285, 3, 4}, {336, 5, 58, 160, 2, 4},  {384, 1, 30, 160, 2, 4},  {385, 1, 30, 160, 1, 8}, {512, 8, 30, 160, 1, 8},
    {513, 8, 30, 160, 2, 4},  {592, 1, 16, 133, 2, 4},  {592, 1, 16, 97, 1, 4},   {912, 2, 50, 128, 1, 4}, {512, 5, 256, 22, 1, 4},
    // above the ceiling of one workgroup a pair those of four are no choice
    {1025, 1, 40, 160, 1, 8}, {1200, 8, 0, 256, 1, 8},
    {1, 1, 40, 125, 11, 4},   {80, 7, 62, 125, 6, 4},   {192, 1, 7, 125, 1, 8},   {264, 8, 3, 125, 1, 4},  {20, 6, 0, 189, 2, 4},
    // the ceiling of 64 workgroups a pair
    {1, 7, 508, 128, 64, 8},  {1, 1, 1024, 128, 64, 8}, {2, 7, 4096, 1, 64, 8},   {3, 1, 600, 20, 64, 8},  {4, 8, 1024, 128, 64, 8},
};

static void different_lengths(std::mt19937& rng) {
  auto below = [&](int n) { return (int)(rng() % (unsigned)n); };
  const int B = 2 + below(1 + below(255)), Hkv = 1 + below(1 + below(32)), most = 1 + below(1 + below(4096)), rows = 32 * (1 + below(12));
  const CacheView v = view_of(B, Hkv, 8);
  SeqCounts sc{};
  sc.enabled = 1;
  int n_blocks = 0, n_fp16 = 0;
  for (int b = 0; b < B; ++b) {
    sc.n_blocks[b] = below(most + 1);
    const uint32_t nf = (uint32_t)below(rows + 1);
    sc.n_fp16[b >> 1] |= nf << (16 * (b & 1));
    n_blocks = sc.n_blocks[b] > n_blocks ? sc.n_blocks[b] : n_blocks;
    n_fp16 = (int)nf > n_fp16 ? (int)nf : n_fp16;
  }
  int ns;
  DecodeGrid dg;
  choose_splits(v, n_blocks, n_fp16, false, &ns, &dg);
  if (dg.n_splits > max_splits_for(v.P)) return;
  deal_by_length(v, dg.n_splits, &sc, &dg);
#define AT "B %d, Hkv %d, up to %d records and %d rows: %d units of %d wavefronts", B, Hkv, most, rows, sc.n_units, dg.n_waves
  if (sc.n_units == 0) {
    CHECK(dg.n_waves == 4, AT);
    return;
  }
  CHECK(sc.n_units <= kMaxUnits && sc.n_units <= B * max_splits_for(v.P), AT);      // (the units' partials fit the workspace)
  CHECK(dg.n_waves == 4 || sc.n_units * Hkv <= 256, AT);      // workgroups of eight in one round
  int at = 0;
  for (int b = 0; b < B; ++b) {
    const int first = (int)(sc.span[b] & 0xffffu), n = (int)(sc.span[b] >> 16);
    CHECK(first == at && n >= 1 && n * dg.n_waves >= (fp16_rows_of(sc, b) + 31) / 32, AT);
    for (int u = first; u < first + n; ++u) CHECK((sc.owner[u >> 2] >> (8 * (u & 3)) & 0xffu) == (unsigned)b, AT);
    at += n;
  }
  CHECK(at == sc.n_units, AT);
#undef AT
}

int main() {
  for (int P = 1; P <= 512; P += P < 40 ? 1 : 1 + P / 16)
    for (int n_blocks = 0; n_blocks <= 4096; n_blocks += n_blocks < 700 ? 1 : 37)
      for (int n_fp16 : {0, 1, 32, 33, 100, 128, 160, 225, 256, 384})
        if (n_blocks + n_fp16 > 0)
          for (int g : {1, 8}) equal_lengths(P, g, n_blocks, n_fp16);
  for (int P : {513, 700, 1023, 1024, 1025, 4096})
    for (int n_blocks = 0; n_blocks <= 300; ++n_blocks)
      for (int n_fp16 : {1, 33, 128, 160, 256, 384}) equal_lengths(P, 8, n_blocks, n_fp16);
  for (const auto& l : kLines) {
    int ns;
    DecodeGrid got;
    choose_splits(view_of(l.P, 1, l.g), l.n_blocks, l.n_fp16, true, &ns, &got);
    CHECK(got.n_splits == l.n_splits && got.n_waves == l.n_waves, "P %d, %d heads, %d records, %d fp16 rows: %d workgroups of %d instead of %d of %d",
          l.P, l.g, l.n_blocks, l.n_fp16, got.n_splits, got.n_waves, l.n_splits, l.n_waves);
  }
  std::mt19937 rng(1);
  for (int i = 0; i < 20000; ++i) different_lengths(rng);
  printf("decode grids: ok\n");
  return 0;
}
