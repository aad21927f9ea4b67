// csrc/api.hip linked against launchers that only take notes and fail on demand: what the host keeps of a decode step whose
// launches fail part-way.  No HIP call reaches a device.
#include <cstdio>
#include <cstdlib>
#include "mixkvq_internal.h"

namespace mixkvq {
static int g_flushes = 0, g_clears = 0, g_attentions = 0;
static bool g_fail_flush = false, g_fail_attention = false;
hipError_t launch_zero_qacc(const CacheView&, hipStream_t) { return ++g_clears, hipSuccess; }
hipError_t launch_zero_tickets(const CacheView&, hipStream_t) { return hipSuccess; }
hipError_t launch_zero_qacc_listed(const CacheView&, const FlushList&, hipStream_t) { return ++g_clears, hipSuccess; }
hipError_t launch_select(const CacheView&, const __half*, int, Strides3, const __half*, int, Strides3, uint8_t*, hipStream_t) {
  return hipSuccess;
}
hipError_t launch_select2(const CacheView&, const __half*, int, Strides3, const __half*, int, Strides3, uint8_t*, hipStream_t) {
  return hipSuccess;
}
uint8_t* select_scratch(const CacheView& v) { return v.ws; }
hipError_t launch_flush(const CacheView&, const __half*, const __half*, Strides3, int, int, int, const uint8_t*, int, hipStream_t) {
  return ++g_flushes, g_fail_flush ? hipErrorUnknown : hipSuccess;
}
hipError_t launch_flush_windows(const CacheView&, const FlushList&, hipStream_t) {
  return ++g_flushes, g_fail_flush ? hipErrorUnknown : hipSuccess;
}
hipError_t launch_residual_copy(const CacheView&, const __half*, const __half*, Strides3, int, int, int, hipStream_t) {
  return hipSuccess;
}
hipError_t launch_decode(const CacheView&, const __half*, __half*, float*, float, int, int, int, NewToken, SeqCounts*, hipStream_t,
                         hipEvent_t, hipEvent_t, int*, float*) {
  return ++g_attentions, g_fail_attention ? hipErrorUnknown : hipSuccess;
}
size_t decode_launch_partials_bytes(const CacheView&, int, int) { return 0; }
hipError_t noalloc_scratch(void**) { return hipErrorUnknown; }
size_t decode_workspace_bytes(const mixkvq_config&) { return 1 << 20; }
size_t select_workspace_bytes(const mixkvq_config&) { return 1 << 20; }
}  // namespace mixkvq

#define CHECK(cond)                                                            \
  do {                                                                         \
    if (!(cond)) {                                                             \
      fprintf(stderr, "%s:%d: check failed: %s\n", __FILE__, __LINE__, #cond); \
      exit(1);                                                                 \
    }                                                                          \
  } while (0)

static bool state_is(mixkvq_cache* c, int b, int64_t nq, int32_t nr) {
  int64_t q;
  int32_t r, s;
  return mixkvq_cache_state_seq(c, b, &q, &r, &s) == MIXKVQ_OK && q == nq && r == nr && s == 0;
}

int main() {
  using namespace mixkvq;
  mixkvq_config cfg{};
  cfg.B = 3; cfg.Hq = 4; cfg.Hkv = 2; cfg.D = 128; cfg.T_max = 512; cfg.Gk = cfg.Gv = cfg.R = 128; cfg.k4 = 16;
  cfg.qacc_reset_on_flush = 1;
  char* const at = (char*)0x100000000000ull;      // (never dereferenced)
  const mixkvq_buffers bufs{at, at + (1ll << 32), at + (2ll << 32), at + (3ll << 32), at + (4ll << 32)};
  const int64_t st[3] = {2 * 128, 128, 128};
  for (int ragged = 0; ragged < 2; ++ragged) {
    mixkvq_cache* c = nullptr;
    CHECK(mixkvq_cache_create(&cfg, &bufs, &c) == MIXKVQ_OK);
    const int third = ragged ? 50 : 128;      // tokens in the window of the third sequence; the others have a full one
    for (int b = 0; b < 3; ++b) CHECK(mixkvq_cache_set_state_seq(c, b, 0, b == 2 ? third : 128, 0) == MIXKVQ_OK);
    auto step = [&] { return mixkvq_decode_step(c, at, at, st, at, at, nullptr, 0.f, 1, nullptr); };
    // the packing fails: nothing has changed
    g_flushes = g_clears = g_attentions = 0;
    g_fail_flush = true;
    CHECK(step() == MIXKVQ_EHIP && g_flushes == 1 && g_attentions == 0);
    CHECK(state_is(c, 0, 0, 128) && state_is(c, 1, 0, 128) && state_is(c, 2, 0, third));
    // the blocks are packed and their accumulators cleared, the attention fails: the blocks stay packed (a second
    // packing would score them with cleared accumulators), the token is not in
    g_flushes = g_clears = g_attentions = 0;
    g_fail_flush = false;
    g_fail_attention = true;
    CHECK(step() == MIXKVQ_EHIP && g_flushes == 1 && g_clears == 1 && g_attentions == 1);
    CHECK(state_is(c, 0, 128, 0) && state_is(c, 1, 128, 0) && (ragged ? state_is(c, 2, 0, 50) : state_is(c, 2, 128, 0)));
    // the same step again
    g_fail_attention = false;
    CHECK(step() == MIXKVQ_OK && g_flushes == 1 && g_clears == 1 && g_attentions == 2);
    CHECK(state_is(c, 0, 128, 1) && state_is(c, 1, 128, 1) && (ragged ? state_is(c, 2, 0, 51) : state_is(c, 2, 128, 1)));
    mixkvq_cache_destroy(c);
  }
  printf("host launch stub: ok\n");
  return 0;
}
