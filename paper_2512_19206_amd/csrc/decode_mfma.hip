// Matrix-core decode attention: the merge kernel and the table of the variants instantiated for the measured
// configurations; decode_mfma_kernel.h holds the kernel itself, decode_mfma_generic_*.hip the wider tables.
#define MIXKVQ_MFMA_MAIN_TU
#include "decode_mfma_generic.h"

namespace mixkvq {

// The merge as a launch of its own, one workgroup per pair, in the order of sums of the attention launch's own (see merge_pair).
__global__ void __launch_bounds__(512)
decode_merge_pair_kernel(CacheView cv, const float* __restrict__ part, int n_parts, int n_half, __half* __restrict__ out,
                         float* __restrict__ lse) {
  __shared__ __align__(16) unsigned char lds[6144];
  const int p = blockIdx.x, tid = threadIdx.x, h = tid >> 5 & 7, g = cv.g;
  const size_t bh = (size_t)(p / cv.cfg.Hkv) * cv.cfg.Hq + (size_t)(p % cv.cfg.Hkv) * g + h;
  merge_pair<false>(part + (size_t)p * n_parts * g * kPartStrideM, n_parts, n_half, tid, g, lds, out, lse, bh, cv.cfg.in_dtype);
}

hipError_t launch_merge_pair(const CacheView& v, const float* part, DecodeGrid dg, __half* out, float* lse, hipStream_t s) {
  decode_merge_pair_kernel<<<dim3(v.P), dim3(64 * dg.n_waves), 0, s>>>(v, part, dg.n_splits, dg.n_waves >> 2, out, lse);
  return hipGetLastError();
}

// Returns true and launches when the configuration is one the matrix-core kernel covers.
bool try_launch_decode_mfma(const CacheView& v, const __half* q, float scale, int n_blocks, int n_res, DecodeGrid dg,
                            float* part, __half* out, float* lse, int accumulate_q, NewToken nt, const SeqCounts& sc,
                            hipStream_t s, hipEvent_t ev_start, hipEvent_t ev_stop, hipError_t* err) {
  const mixkvq_config& c = v.cfg;
  // key groups of 32 tokens take the G32 variants, multiples of 64 the others; value groups of 32, 64 or 128 channels
  // records of 32 tokens (one key group each) take the RH variants
  // A cache that holds fp16 rows only (n_blocks == 0, the first answers after a short prompt) runs here as well: one
  // launch that moves the new token, adds |q| and attends, 9.4 us per step of one 28/4-head sequence of 90 tokens
  // against 19.2 us for the vector-ALU path's four launches, with the same outputs to 1.1e-6 (the fp16 rows' weights keep
  // their binary16 remainder; rounded to binary16 alone the outputs were 1.1e-4 apart).
  const int rh = c.R == 32 && c.Gk == 32;
  if ((c.R % 64 != 0 && !rh) || (c.Gk % 64 != 0 && c.Gk != 32) || (c.Gv % 64 != 0 && c.Gv != 32)) return false;
  // (queries that do not start on 8 bytes, which this kernel reads at a time, stay with the vector-ALU path there)
  if (n_blocks < 1 && (reinterpret_cast<uintptr_t>(q) & 7u)) return false;
  if (v.lay.off_v > kKPartMax || v.lay.rec_bytes - v.lay.off_v_s > kVMetaMax) return false;
  const int nvg = v.lay.NVG;
  const int nkl = (v.lay.off_v / 16 + 63) / 64;
  const int g32 = c.Gk == 32 && !rh;
  const int paged = v.table != nullptr;
  hipError_t e = hipErrorInvalidValue;
  bool ok = true;
#define MIXKVQ_CASE(K4_, K16_, NVG_, NKL_, RG_, THR_, G32_, PG_, RH_)                                               \
  if (c.k4 == K4_ && c.k16 == K16_ && nvg == NVG_ && nkl <= NKL_ && c.policy == THR_ && g32 == G32_ && paged == PG_ && \
      rh == RH_ && (RG_ != 2 || dg.streamed) && (RG_ == 0 || (c.R == 128 && c.Gk == 128 && HalfSplit<K4_, K16_, THR_>::off_klo == v.lay.off_klo &&  \
                                 HalfSplit<K4_, K16_, THR_>::off_k4 == v.lay.off_k4 &&                              \
                                 HalfSplit<K4_, K16_, THR_>::off_k16 == v.lay.off_k16 &&                            \
                                 HalfSplit<K4_, K16_, THR_>::off_v == v.lay.off_v)))                                \
    e = launch_one<K4_, K16_, NVG_, NKL_, RG_, THR_, G32_, PG_, RH_>(v, q, scale, n_blocks, n_res, dg, part, out, lse,  \
                                                           accumulate_q, nt, sc, s, ev_start, ev_stop);             \
  else
  MIXKVQ_CASE(16, 0, 1, 6, 2, 0, 0, 0, 0)
  MIXKVQ_CASE(0, 12, 1, 8, 2, 0, 0, 0, 0)
  MIXKVQ_CASE(8, 0, 1, 6, 2, 0, 0, 0, 0)
  MIXKVQ_CASE(16, 0, 1, 6, 1, 0, 0, 0, 0)
  MIXKVQ_CASE(0, 12, 1, 8, 1, 0, 0, 0, 0)
  MIXKVQ_CASE(8, 0, 1, 6, 1, 0, 0, 0, 0)
  MIXKVQ_CASE(16, 0, 1, 6, 0, 0, 0, 0, 0)
  MIXKVQ_CASE(0, 12, 1, 8, 0, 0, 0, 0, 0)
  MIXKVQ_CASE(0, 0, 1, 6, 0, 0, 0, 0, 0)
  MIXKVQ_CASE(8, 0, 1, 6, 0, 0, 0, 0, 0)
  MIXKVQ_CASE(24, 0, 1, 6, 0, 0, 0, 0, 0)
  MIXKVQ_CASE(32, 0, 1, 6, 0, 0, 0, 0, 0)
  MIXKVQ_CASE(16, 0, 2, 6, 0, 0, 0, 0, 0)
  MIXKVQ_CASE(0, 12, 2, 8, 0, 0, 0, 0, 0)
  MIXKVQ_CASE(8, 4, 1, 8, 0, 0, 0, 0, 0)
  MIXKVQ_CASE(0, 32, 1, 12, 0, 0, 0, 0, 0)
  MIXKVQ_CASE(0, 4, 1, 6, 0, 0, 0, 0, 0)
  MIXKVQ_CASE(0, 8, 1, 7, 0, 0, 0, 0, 0)
  MIXKVQ_CASE(0, 16, 1, 8, 0, 0, 0, 0, 0)
  MIXKVQ_CASE(0, 24, 1, 10, 0, 0, 0, 0, 0)
  MIXKVQ_CASE(16, 4, 1, 8, 0, 0, 0, 0, 0)
  MIXKVQ_CASE(16, 8, 1, 8, 0, 0, 0, 0, 0)
  // threshold policy: the capacities of the two side tiers
  MIXKVQ_CASE(16, 8, 1, 8, 0, 1, 0, 0, 0)
  MIXKVQ_CASE(16, 0, 1, 6, 0, 1, 0, 0, 0)
  MIXKVQ_CASE(0, 12, 1, 8, 0, 1, 0, 0, 0)
  MIXKVQ_CASE(8, 4, 1, 8, 0, 1, 0, 0, 0)
  // key groups of 32 tokens
  MIXKVQ_CASE(16, 0, 1, 7, 0, 0, 1, 0, 0)
  MIXKVQ_CASE(8, 0, 1, 7, 0, 0, 1, 0, 0)
  MIXKVQ_CASE(0, 0, 1, 7, 0, 0, 1, 0, 0)
  MIXKVQ_CASE(16, 0, 2, 7, 0, 0, 1, 0, 0)
  MIXKVQ_CASE(16, 0, 1, 8, 0, 1, 1, 0, 0)
  // value groups of 32 channels (with key groups of 32 tokens: the group size of the paper's experiments)
  MIXKVQ_CASE(0, 12, 4, 10, 0, 0, 1, 0, 0)
  MIXKVQ_CASE(0, 8, 4, 10, 0, 0, 1, 0, 0)
  MIXKVQ_CASE(16, 8, 4, 10, 0, 1, 1, 0, 0)
  MIXKVQ_CASE(0, 12, 4, 10, 0, 1, 1, 0, 0)
  MIXKVQ_CASE(8, 4, 4, 10, 0, 0, 1, 0, 0)
  MIXKVQ_CASE(0, 12, 1, 10, 0, 0, 1, 0, 0)
  MIXKVQ_CASE(16, 8, 1, 10, 0, 1, 1, 0, 0)
  MIXKVQ_CASE(0, 12, 1, 10, 0, 1, 1, 0, 0)
  MIXKVQ_CASE(16, 16, 4, 12, 0, 1, 1, 0, 0)
  MIXKVQ_CASE(16, 0, 4, 7, 0, 0, 1, 0, 0)
  MIXKVQ_CASE(8, 0, 4, 7, 0, 0, 1, 0, 0)
  MIXKVQ_CASE(16, 0, 4, 8, 0, 1, 1, 0, 0)
  MIXKVQ_CASE(16, 0, 4, 6, 0, 0, 0, 0, 0)
  // paged layout (block table): the main tiers
  MIXKVQ_CASE(16, 0, 1, 6, 0, 0, 0, 1, 0)
  MIXKVQ_CASE(0, 12, 1, 8, 0, 0, 0, 1, 0)
  MIXKVQ_CASE(8, 0, 1, 6, 0, 0, 0, 1, 0)
  MIXKVQ_CASE(16, 8, 1, 8, 0, 1, 0, 1, 0)
  MIXKVQ_CASE(16, 0, 4, 7, 0, 0, 1, 1, 0)
  MIXKVQ_CASE(16, 8, 4, 10, 0, 1, 1, 1, 0)
  // records of 32 tokens (the shorter residual length of the paper's throughput runs), value groups of 32 or 128 channels
  MIXKVQ_CASE(16, 0, 4, 2, 0, 0, 0, 0, 1)
  MIXKVQ_CASE(8, 0, 4, 2, 0, 0, 0, 0, 1)
  MIXKVQ_CASE(0, 0, 4, 2, 0, 0, 0, 0, 1)
  MIXKVQ_CASE(16, 0, 1, 2, 0, 0, 0, 0, 1)
  MIXKVQ_CASE(8, 4, 4, 2, 0, 0, 0, 0, 1)
  MIXKVQ_CASE(16, 8, 4, 3, 0, 1, 0, 0, 1)
  MIXKVQ_CASE(16, 0, 4, 3, 0, 1, 0, 0, 1)
  ok = false;
#undef MIXKVQ_CASE
  if (!ok) {     // not one of the variants above: the wider tables (they take either layout)
    const GenericArgs a{v, q, scale, n_blocks, n_res, dg, part, out, lse, accumulate_q, nt, sc, s, ev_start, ev_stop,
                        nkl, g32, rh};
    return rh ? try_launch_generic_rh(a, err) : (g32 ? try_launch_generic_g32(a, err) : try_launch_generic_plain(a, err));
  }
  *err = e;
  return true;
}

}  // namespace mixkvq

#ifdef MIXKVQ_PHASE_CLOCKS
extern "C" int mixkvq_debug_phase_clocks(void* host_dst, size_t bytes) {
  (void)hipDeviceSynchronize();
  return (int)hipMemcpyFromSymbol(host_dst, HIP_SYMBOL(mixkvq::g_phase_clock), bytes);
}
#endif
