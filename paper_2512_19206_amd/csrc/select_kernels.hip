// Channel-salience statistics and top-k selection (Section 4.2, Eq. 6-8).
//
// Everything that decides an index is exact: |q| sums and key ranges are integers
// in units of 2^-24 (every finite fp16 is a multiple of it), so the reductions may
// run in any order; the score is one binary64 product.
#include "mixkvq_internal.h"

namespace mixkvq {

// ---------------------------------------------------------------------------
// accumulator clear
// ---------------------------------------------------------------------------
__global__ void zero_u64_kernel(unsigned long long* sums, size_t n_sums, unsigned long long* counts, size_t n_counts) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n_sums) sums[i] = 0ull;
  else if (i < n_sums + n_counts) counts[i - n_sums] = 0ull;
}

// the sums and the counts of the view's pairs (two ranges: a view of some sequences of the batch is not contiguous)
hipError_t launch_zero_qacc(const CacheView& v, hipStream_t s) {
  const size_t n_sums = (size_t)v.P * kD, n = n_sums + (size_t)v.P;
  zero_u64_kernel<<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s>>>(v.qacc, n_sums, v.qcnt, (size_t)v.P);
  return hipGetLastError();
}

// One workgroup per pair of the listed sequences.  (A launch per sequence: 411 us for a step in which 255 of 256 sequences
// pack a block, 24 this way.)
__global__ void __launch_bounds__(kD) zero_listed_kernel(CacheView cv, FlushList list) {
  const int Hkv = cv.cfg.Hkv, p = (int)list.seq[blockIdx.x / Hkv] * Hkv + blockIdx.x % Hkv;
  cv.qacc[(size_t)p * kD + threadIdx.x] = 0ull;
  if (threadIdx.x == 0) cv.qcnt[p] = 0ull;
}

hipError_t launch_zero_tickets(const CacheView& v, hipStream_t s) {
  zero_u64_kernel<<<dim3((unsigned)((v.P + 255) / 256)), dim3(256), 0, s>>>(v.tickets, (size_t)v.P, nullptr, 0);
  return hipGetLastError();
}

hipError_t launch_zero_qacc_listed(const CacheView& v, const FlushList& list, hipStream_t s) {
  zero_listed_kernel<<<dim3(list.n * v.cfg.Hkv), dim3(kD), 0, s>>>(v, list);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Scoring and selection in one launch.  Workgroups (pair, y): the first nq of a pair add |q| (Eq. 6) over one piece of
// one query head each, the others take the range (Eq. 7) of one piece of the keys; the last of a pair to finish scores
// and selects (Eq. 8).  Memory-bound on large tensors: 16 threads cover a row of 256 bytes with one 16-byte load each,
// 16 rows per pass, eight passes in flight.
//   |q|     per-thread sums, one LDS reduction over the 16 row lanes, one 64-bit atomic per channel and workgroup
//           (integers: any order is exact).
//   range   running minima and maxima of packed 16-bit keys that order like the fp16 values; a workgroup leaves its
//           result (128 channels, 512 bytes) in the workspace, so nothing has to be initialised.
//   select  the workgroups of a pair draw tickets.  Sums, partial ranges and tickets are agent-scope accesses (they pass
//           the chip's eight L2 caches by), and a workgroup's own have been acknowledged before its ticket is drawn.
// As launches of their own (|q|, initial ranges, ranges, selection) the four took 7.5 + 1.4 + 6.3 + 9.5 us and the gaps
// between them on 8 pairs of 1 000 tokens, of which the work itself is a fraction.
// ---------------------------------------------------------------------------
constexpr int kStreamThreads = 256;
constexpr int kMinRowsPerWG = 256, kMaxRowsPerWG = 8192;
constexpr int kMaxExactRows = 131072;      // rows of a |q| workgroup up to which its binary64 sums are exact
constexpr int kInFlight = 8;      // 16-byte loads a thread has in flight
constexpr int kRangePartBytes = kD * 4;    // partial range of one workgroup: 64 words of minima, 64 of maxima

struct SelectArgs {
  const __half *q, *kA, *kB;       // queries; keys: run A (binary16 window rows), then run B (the caller's tensor)
  Strides3 qs, sA, sB;
  int Lq, LA, LB;
  int rows_q, rows_k;              // rows one workgroup takes
  int nq, nA, nB;                  // workgroups per pair
  unsigned* part;                  // [P][nA + nB][128]
  uint8_t* sel;                    // [P][k16 + k4]
};

// Rows one workgroup takes.  Small calls are bound by latency: 256 rows are two passes of eight loads (128 and 512: 35.4
// and 34.7 us for a prompt of 1 531 tokens in 4 pairs, 256: 33.2).  More rows as soon as that still leaves every compute
// unit four workgroups, and above 512 rows eight of them: fewer reductions, atomics and tickets per byte streamed (16
// prompts of 32 768 tokens, up to 2 048 / 4 096 / 8 192 rows: 1 810, 1 775, 1 742 us; 32 768 rows measure the same).
static int rows_per_workgroup(int64_t pairs_times_heads, int L) {
  int rows = kMinRowsPerWG;
  while (rows < kMaxRowsPerWG &&
         pairs_times_heads * (((int64_t)L + 2 * rows - 1) / (2 * rows)) >= (rows < 512 ? 1024 : 2048)) rows *= 2;
  return rows;
}

typedef short s16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ s16x2 order_key(unsigned w) {     // involution: also maps keys back to fp16 bits
  const s16x2 v = __builtin_bit_cast(s16x2, w);
  return v ^ ((v >> 15) & (short)0x7fff);
}
__device__ __forceinline__ s16x2 as_key(unsigned w) { return __builtin_bit_cast(s16x2, w); }

// The per-thread sums run in binary64, which is exact here: every |fp16| is a multiple of 2^-24 below 2^16, so up to
// 2^13 of them add without rounding in a 53-bit significand (a thread adds rows / 16 per channel);
// the sum times 2^24 is the exact integer.
typedef _Float16 sh2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void add8(double (&acc)[8], uint4 v) {
  const unsigned w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const sh2 h = __builtin_bit_cast(sh2, w[i]);
    acc[2 * i] += __builtin_fabs((double)(float)h[0]);
    acc[2 * i + 1] += __builtin_fabs((double)(float)h[1]);
  }
}

// eight elements of a row; rows of any alignment when AL is false; NT: with the non-temporal policy (aligned rows)
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
template <bool AL, bool NT>
__device__ __forceinline__ uint4 load8(const __half* p) {
  if (AL && NT) return __builtin_bit_cast(uint4, __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p)));
  if (AL) return *reinterpret_cast<const uint4*>(p);
  unsigned w[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) w[i] = (unsigned)h2bits(p[2 * i]) | ((unsigned)h2bits(p[2 * i + 1]) << 16);
  return make_uint4(w[0], w[1], w[2], w[3]);
}

// f(16-byte piece) for rows t0 + r, t0 + r + 16, ... below t1; `base` is this thread's piece of row 0
template <bool AL, bool NT, class F>
__device__ __forceinline__ void stream_rows(const __half* base, int64_t stride_t, int t0, int t1, int r, bool bf16, F f) {
  int t = t0 + r;
  constexpr int NF = kInFlight;
  for (; t + 16 * (NF - 1) < t1; t += 16 * NF) {
    uint4 v[NF];
#pragma unroll
    for (int u = 0; u < NF; ++u) v[u] = load8<AL, NT>(base + (int64_t)(t + 16 * u) * stride_t);
#pragma unroll
    for (int u = 0; u < NF; ++u) f(as_f16x8(v[u], bf16));
  }
  if (t < t1) {      // up to seven rows more: asked for together as well (a row past the end repeats the last one)
    uint4 v[NF - 1];
#pragma unroll
    for (int u = 0; u < NF - 1; ++u) v[u] = load8<AL, NT>(base + (int64_t)(t + 16 * u < t1 ? t + 16 * u : t) * stride_t);
#pragma unroll
    for (int u = 0; u < NF - 1; ++u)
      if (t + 16 * u < t1) f(as_f16x8(v[u], bf16));
  }
}

template <class T>
__device__ __forceinline__ T load_agent(const T* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// BF: the caller's tensors hold bfloat16 (converted to binary16 on entry); AL: 16-byte aligned rows.
// The queries are read once, with the non-temporal policy, so that the keys stay in the last-level cache (256 MB) for the pack
// kernel that follows.  us without / queries / queries and keys: 4 prompts of 5 000 tokens (41 MB of keys) 88.5 / 79.5 / 81.6,
// 9 chunks of 1 000 in 2 sequences 217 / 210 / 220, 16 prompts of 32 768 (1 GB) 1 764 / 1 668 / 1 656.
template <bool BF, bool AL>
__global__ void __launch_bounds__(kStreamThreads) select_kernel(CacheView cv, SelectArgs a) {
  __shared__ __align__(16) unsigned char smem[16 * kD * 8];
  __shared__ int sTicket;
  __shared__ unsigned long long sCount;
  const int Hkv = cv.cfg.Hkv, g = cv.g;
  const int p = blockIdx.x, b = p / Hkv, j = p % Hkv, tid = threadIdx.x, y = blockIdx.y;
  const int c = tid & 15, r = tid >> 4;
  const int nk = a.nA + a.nB;
  // The pair's token count, which its last workgroup advances; only thresholds look at it (read ahead then: behind the ticket
  // that cost 0.7 us of 8; added by every |q| workgroup beside its ticket, 2 of 12).
  const unsigned long long added = (unsigned long long)a.Lq * (unsigned long long)g;
  unsigned long long count = 0ull;
  if (tid == 0 && cv.cfg.policy == 1) count = cv.qcnt[p] + added;
  if (y < a.nq) {
    auto sAcc = reinterpret_cast<unsigned long long (*)[kD]>(smem);      // [16][kD]
    const int hh = y % g, t0 = (y / g) * a.rows_q, t1 = min(a.Lq, t0 + a.rows_q);
    double acc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = 0.0;
    stream_rows<AL, true>(a.q + (int64_t)b * a.qs.b + (int64_t)(j * g + hh) * a.qs.h + 8 * c, a.qs.t, t0, t1, r, BF,
                    [&](uint4 v) { add8(acc, v); });
#pragma unroll
    for (int i = 0; i < 8; ++i) sAcc[r][8 * c + i] = (unsigned long long)(acc[i] * 16777216.0);
    __syncthreads();
    if (tid < kD) {
      unsigned long long sum = 0;
#pragma unroll
      for (int rr = 0; rr < 16; ++rr) sum += sAcc[rr][tid];
      __hip_atomic_fetch_add(cv.qacc + (size_t)p * kD + tid, sum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  } else {
    auto sLo = reinterpret_cast<unsigned (*)[kD / 2]>(smem);      // [16][kD / 2]
    auto sHi = sLo + 16;
    const int yk = y - a.nq;
    const bool inA = yk < a.nA;
    const Strides3 ks = inA ? a.sA : a.sB;
    const int L = inA ? a.LA : a.LB, t0 = (inA ? yk : yk - a.nA) * a.rows_k, t1 = min(L, t0 + a.rows_k);
    s16x2 lo[4], hi[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      lo[i] = s16x2{(short)0x7fff, (short)0x7fff};
      hi[i] = s16x2{(short)-0x8000, (short)-0x8000};
    }
    stream_rows<AL, false>((inA ? a.kA : a.kB) + (int64_t)b * ks.b + (int64_t)j * ks.h + 8 * c, ks.t, t0, t1, r, BF && !inA,
                    [&](uint4 v) {
                      const unsigned w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                      for (int i = 0; i < 4; ++i) {
                        const s16x2 key = order_key(w[i]);
                        lo[i] = __builtin_elementwise_min(lo[i], key);
                        hi[i] = __builtin_elementwise_max(hi[i], key);
                      }
                    });
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      sLo[r][4 * c + i] = __builtin_bit_cast(unsigned, lo[i]);
      sHi[r][4 * c + i] = __builtin_bit_cast(unsigned, hi[i]);
    }
    __syncthreads();
    if (tid < kD) {      // the first wavefront joins the minima, the second the maxima
      const int d2 = tid & 63;
      s16x2 m = as_key(tid < 64 ? sLo[0][d2] : sHi[0][d2]);
#pragma unroll
      for (int rr = 1; rr < 16; ++rr)
        m = tid < 64 ? __builtin_elementwise_min(m, as_key(sLo[rr][d2])) : __builtin_elementwise_max(m, as_key(sHi[rr][d2]));
      __hip_atomic_store(a.part + ((size_t)p * nk + yk) * kD + tid, __builtin_bit_cast(unsigned, m), __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  // every store and atomic of this workgroup has reached the coherence point before its ticket is drawn
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (tid == 0) {
    sTicket = (int)__hip_atomic_fetch_add(cv.tickets + p, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    sCount = count;
  }
  __syncthreads();
  if (sTicket != a.nq + nk - 1) return;
  // ---- the pair's last workgroup: all sums and partial ranges are there; the ticket goes back to 0 ----
  if (tid == 0) {
    __hip_atomic_fetch_sub(cv.tickets + p, (unsigned long long)(a.nq + nk), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (added) __hip_atomic_fetch_add(cv.qcnt + p, added, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  unsigned long long sum = 0ull;
  if (tid < kD) sum = load_agent(cv.qacc + (size_t)p * kD + tid);
  {
    const unsigned* part = a.part + (size_t)p * nk * kD + (tid & 63);
    s16x2 lo = s16x2{(short)0x7fff, (short)0x7fff}, hi = s16x2{(short)-0x8000, (short)-0x8000};
    constexpr int NF = 8;
    for (int i0 = tid >> 6; i0 < nk; i0 += 4 * NF) {
      unsigned vl[NF], vh[NF];
#pragma unroll
      for (int u = 0; u < NF; ++u) {
        const size_t at = (size_t)(i0 + 4 * u < nk ? i0 + 4 * u : i0) * kD;
        vl[u] = load_agent(part + at);
        vh[u] = load_agent(part + at + 64);
      }
#pragma unroll
      for (int u = 0; u < NF; ++u) {
        lo = __builtin_elementwise_min(lo, as_key(vl[u]));
        hi = __builtin_elementwise_max(hi, as_key(vh[u]));
      }
    }
    unsigned* sM = reinterpret_cast<unsigned*>(smem);      // [4][2][64]
    sM[tid >> 6 << 7 | (tid & 63)] = __builtin_bit_cast(unsigned, order_key(__builtin_bit_cast(unsigned, lo)));
    sM[tid >> 6 << 7 | 64 | (tid & 63)] = __builtin_bit_cast(unsigned, order_key(__builtin_bit_cast(unsigned, hi)));
  }
  __syncthreads();
  double* sA = reinterpret_cast<double*>(smem + 2048);
  unsigned* sPart = reinterpret_cast<unsigned*>(smem + 2048 + 1024);
  if (tid < kD) {
    const unsigned short* m = reinterpret_cast<const unsigned short*>(smem);      // [4][2][128] fp16 bits
    long long lo = fix24(m[tid]), hi = fix24(m[kD + tid]);
#pragma unroll
    for (int w = 1; w < 4; ++w) {
      const long long l = fix24(m[2 * kD * w + tid]), h = fix24(m[2 * kD * w + kD + tid]);
      lo = l < lo ? l : lo;
      hi = h > hi ? h : hi;
    }
    const long long rng = hi - lo;
    sA[tid] = cv.cfg.score_mode ? (double)rng : (double)sum * (double)rng;
  }
  __syncthreads();
  const int tier = rank_channels<kStreamThreads>(cv.cfg, sCount, sA, sPart);      // (threads 0..127: of their channel)
  // positions inside the tiers: ballots over the two wavefronts that hold the channels
  const unsigned long long m1 = __ballot(tier == 1), m2 = __ballot(tier == 2);
  unsigned long long* sMask = reinterpret_cast<unsigned long long*>(smem);      // the first wavefront's two ballots
  if (tid == 0) sMask[0] = m1, sMask[1] = m2;
  __syncthreads();
  const int k16 = cv.cfg.k16, k4 = cv.cfg.k4, ks = k16 + k4;
  uint8_t* out = a.sel + (size_t)p * ks;
  const bool second = tid >= 64;
  const int f1 = second ? __popcll(sMask[0]) : 0, f2 = second ? __popcll(sMask[1]) : 0;
  if (tid < kD && tier) {
    const unsigned long long mine = tier == 2 ? m2 : m1;
    const int pos = __popcll(mine & ((1ull << (tid & 63)) - 1ull)) + (tier == 2 ? f2 : f1);
    out[(tier == 2 ? 0 : k16) + pos] = (uint8_t)tid;
  }
  // entries no channel claims (threshold policy): the second wavefront knows both ballots
  if (second && tid < kD) {
    const int n2 = f2 + __popcll(m2), n1 = f1 + __popcll(m1);
    for (int i = tid - 64; i < ks; i += 64)
      if (i < k16 ? i >= n2 : i - k16 >= n1) out[i] = MIXKVQ_NO_CHANNEL;
  }
}

static bool rows_aligned16(const void* ptr, Strides3 st) {
  return (reinterpret_cast<uintptr_t>(ptr) & 15u) == 0 && st.b % 8 == 0 && st.h % 8 == 0 && st.t % 8 == 0;
}

// The workspace holds a selection per pair (select_scratch), then the partial ranges.
size_t select_workspace_bytes(const mixkvq_config& c) {
  return (size_t)c.B * c.Hkv * kD * 2 * sizeof(long long) + (size_t)c.B * c.Hkv * kD;
}

uint8_t* select_scratch(const CacheView& v) { return v.ws; }

static hipError_t launch_select_kernel(const CacheView& v, SelectArgs a, hipStream_t s) {
  a.rows_q = rows_per_workgroup((int64_t)v.P * v.g, a.Lq);
  auto pieces = [](int L, int rows) { return (int)(((int64_t)L + rows - 1) / rows); };
  while ((int64_t)v.g * pieces(a.Lq, a.rows_q) > 32768 && a.rows_q < kMaxExactRows) a.rows_q *= 2;
  a.nq = v.g * pieces(a.Lq, a.rows_q);
  a.part = reinterpret_cast<unsigned*>(v.ws + (size_t)v.P * kD);
  // as many partial ranges as the workspace has room for (at least four per pair), and as the grid takes
  int64_t room = (v.ws_bytes - (int64_t)v.P * kD) / ((int64_t)v.P * kRangePartBytes);
  room = room < 16384 ? room : 16384;
  int64_t rows = rows_per_workgroup(v.P, a.LA + a.LB);
  while (((int64_t)a.LA + rows - 1) / rows + ((int64_t)a.LB + rows - 1) / rows > room) rows *= 2;
  a.rows_k = (int)(rows < (1ll << 30) ? rows : (1ll << 30));
  a.nA = pieces(a.LA, a.rows_k);
  a.nB = pieces(a.LB, a.rows_k);
  if (a.nq + a.nA + a.nB > 65535) return hipErrorInvalidConfiguration;
  const dim3 grid(v.P, a.nq + a.nA + a.nB), block(kStreamThreads);
  const bool al = (a.nq == 0 || rows_aligned16(a.q, a.qs)) && (a.nB == 0 || rows_aligned16(a.kB, a.sB));
  if (v.cfg.in_dtype) {
    if (al) select_kernel<true, true><<<grid, block, 0, s>>>(v, a);
    else select_kernel<true, false><<<grid, block, 0, s>>>(v, a);
  } else {
    if (al) select_kernel<false, true><<<grid, block, 0, s>>>(v, a);
    else select_kernel<false, false><<<grid, block, 0, s>>>(v, a);
  }
  return hipGetLastError();
}

hipError_t launch_select2(const CacheView& v, const __half* kA, int LA, Strides3 sA, const __half* kB, int LB, Strides3 sB,
                          uint8_t* sel, hipStream_t s) {
  SelectArgs a{};
  a.kA = kA, a.sA = sA, a.LA = LA;
  a.kB = kB, a.sB = sB, a.LB = LB;
  a.sel = sel;
  return launch_select_kernel(v, a, s);
}

hipError_t launch_select(const CacheView& v, const __half* q, int Lq, Strides3 qs, const __half* k, int L, Strides3 ks,
                         uint8_t* sel, hipStream_t s) {
  SelectArgs a{};
  a.q = q, a.qs = qs, a.Lq = Lq;
  a.kB = k, a.sB = ks, a.LB = L;
  a.sel = sel;
  return launch_select_kernel(v, a, s);
}

}  // namespace mixkvq
