// The variants instantiated for the measured configurations, for sequences of equal lengths (Counts = NoCounts) or of any
// lengths (SeqCounts); each is a translation unit of its own.
#pragma once
#include "decode_mfma_generic.h"

namespace mixkvq {

// Launches the variant of the table if the cache is of its kind.
template <class Counts>
static bool try_main_table(const GenericArgs& a, hipError_t* err) {
  const mixkvq_config& c = a.v.cfg;
  const int nvg = a.v.lay.NVG, paged = a.v.table != nullptr;
#define MIXKVQ_CASE(K4_, K16_, NVG_, NKL_, RG_, THR_, G32_, PG_, RH_)                                               \
  if (c.k4 == K4_ && c.k16 == K16_ && nvg == NVG_ && a.nkl <= NKL_ && c.policy == THR_ && a.g32 == G32_ && paged == PG_ && \
      a.rh == RH_ && (RG_ != 2 || a.dg.streamed) && (RG_ == 0 || (c.R == 128 && c.Gk == 128 && HalfSplit<K4_, K16_, THR_>::off_klo == a.v.lay.off_klo &&  \
                                 HalfSplit<K4_, K16_, THR_>::off_k4 == a.v.lay.off_k4 &&                              \
                                 HalfSplit<K4_, K16_, THR_>::off_k16 == a.v.lay.off_k16 &&                            \
                                 HalfSplit<K4_, K16_, THR_>::off_v == a.v.lay.off_v)))                                \
    *err = launch_one<K4_, K16_, NVG_, NKL_, RG_, THR_, G32_, PG_, RH_, Counts>(a.v, a.q, a.scale, a.n_blocks, a.n_res, a.dg, a.part, \
                                                           a.out, a.lse, a.accumulate_q, a.nt, a.sc, a.s, a.ev_start, a.ev_stop);     \
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
  return false;
#undef MIXKVQ_CASE
  return true;
}

}  // namespace mixkvq
