// Matrix-core decode attention: the merge kernel, the choice of a variant and those for sequences of equal lengths;
// decode_mfma_kernel.h holds the kernel itself, decode_mfma_generic_*.hip the wider tables.
#define MIXKVQ_MFMA_MAIN_TU
#include "decode_mfma_table.h"

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

template <class Counts>
static hipError_t launch_rows_only(const GenericArgs& a) {
  return launch_one<0, 0, 1, 1, 3, 0, 0, 0, 0, Counts>(a.v, a.q, a.scale, a.n_blocks, a.n_res, a.dg, a.part, a.out, a.lse,
                                                       a.accumulate_q, a.nt, a.sc, a.s, a.ev_start, a.ev_stop);
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
  const int nkl = (v.lay.off_v / 16 + 63) / 64;
  const int g32 = c.Gk == 32 && !rh;
  const GenericArgs a{v, q, scale, n_blocks, n_res, dg, part, out, lse, accumulate_q, nt, sc, s, ev_start, ev_stop,
                      nkl, g32, rh};
  if (n_blocks < 1) {      // fp16 rows only: one variant for every configuration
    *err = sc.enabled ? launch_rows_only<SeqCounts>(a) : launch_rows_only<NoCounts>(a);
    return true;
  }
  if (sc.enabled ? try_main_table_any_lengths(a, err) : try_main_table<NoCounts>(a, err)) return true;
  // not one of the variants above: the wider tables (they take either layout and any lengths)
  return rh ? try_launch_generic_rh(a, err) : (g32 ? try_launch_generic_g32(a, err) : try_launch_generic_plain(a, err));
}

}  // namespace mixkvq

#ifdef MIXKVQ_PHASE_CLOCKS
extern "C" int mixkvq_debug_phase_clocks(void* host_dst, size_t bytes) {
  (void)hipDeviceSynchronize();
  return (int)hipMemcpyFromSymbol(host_dst, HIP_SYMBOL(mixkvq::g_phase_clock), bytes);
}
#endif
