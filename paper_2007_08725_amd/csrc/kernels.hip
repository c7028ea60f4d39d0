// Device kernels of liblda for gfx950 (CDNA4, wave64).
//
// One synchronous iteration (Sec. 2.2, 3.2, 4.3):
//   k_begin      den[k] = T[k] + V*beta; scheduler counters reset
//   k_topic_list, k_word_pre_small, k_word_pre_wave
//                per word: top-3 of W^[v] (K1, K2, a1..a3), Q' and sum W^   (step 1, Sec. 3.2)
//   k_clear_skips
//                the skip bitmap (one bit per word-ordered token) cleared
//   k_doc_pass   per document: C1, C2 by lookup in the D row, u, M, S_est
//                and the skip test; sets the bit of every skipped token    (steps 2-3, Sec. 3.3)
//   k_sampler (from K = 2,300 on k_sampler_f...), k_sampler_light
//                per unit of a word: W^ row and Q' block prefix in LDS,
//                then for every token whose bit is clear C1 and S' over
//                nz(D[d]) and the final draw over [K1 | S' | Q']; every
//                topic slot of the region written (K1 for the skipped)     (steps 4-6, Sec. 4.3)
//   k_zero_split, k_rebuild_w_wave, k_rebuild_d
//                count tables of the new assignment: dense rows of W by
//                histogram (integer atomics for split words), sparse rows of
//                W and rows of D as packed (topic << 16 | count) entries, T
//                                                                          (Sec. 4.2-4.3)
// The draws are those of fp64 arithmetic (IEEE divide for W^, built without
// contraction); k_sampler_f... and the skip test use single precision where a
// bound proves the fp64 decision.
#include "lda_internal.h"

#include <mutex>

namespace lda {
namespace {

constexpr int kWave = 64;
constexpr int kGroup = 16;  // lanes that cooperate on one token in the sampler
constexpr uint32_t kGroupMask = (1u << kGroup) - 1u;

// ------------------------------------------------------------- Philox ----
// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11): ten rounds of
//   (c0, c1, c2, c3) -> (hi(M1*c2) ^ c1 ^ k0, lo(M1*c2), hi(M0*c0) ^ c3 ^ k1, lo(M0*c0))
// with the key bumped by the Weyl constants between rounds.
__device__ __forceinline__ uint4 philox4x32_10(uint4 c, uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int round = 0; round < 10; ++round) {
    const uint64_t p0 = uint64_t(0xD2511F53u) * c.x, p1 = uint64_t(0xCD9E8D57u) * c.z;  // one 32x32->64 product each
    const uint32_t lo0 = uint32_t(p0), hi0 = uint32_t(p0 >> 32);
    const uint32_t lo1 = uint32_t(p1), hi1 = uint32_t(p1 >> 32);
    c = make_uint4(hi1 ^ c.y ^ k0, lo1, hi0 ^ c.w ^ k1, lo0);
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  return c;
}

// u in [0,1) for token i (input order) at iteration t: counter (i, 0, t, 0).
// The key and t pass through an empty asm so that the compiler computes the
// key schedule where the draw is made instead of keeping twenty hoisted
// round keys live (in the sampler they would spill).
__device__ __forceinline__ double uniform_draw(uint64_t seed, uint32_t t, uint32_t i) {
  uint32_t k0 = uint32_t(seed), k1 = uint32_t(seed >> 32);
  asm volatile("" : "+s"(k0), "+s"(k1), "+s"(t));
  const uint4 x = philox4x32_10(make_uint4(i, 0u, t, 0u), k0, k1);
  const uint64_t bits = (uint64_t(x.x) << 32) | uint64_t(x.y);
  return double(bits >> 11) * 0x1p-53;
}

// W^[v][k] exactly as the paper defines it: an IEEE fp64 divide.
__device__ __forceinline__ double what(uint32_t count, double beta, double den) { return (double(count) + beta) / den; }

// -------------------------------------------------- wave / group helpers --
template <int W>
__device__ __forceinline__ double group_sum(double v) {
#pragma unroll
  for (int o = W / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, W);
  return v;
}

template <int W>
__device__ __forceinline__ uint32_t group_sum_u32(uint32_t v) {
#pragma unroll
  for (int o = W / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, W);
  return v;
}

template <int W>
__device__ __forceinline__ unsigned long long group_sum_u64(unsigned long long v) {
#pragma unroll
  for (int o = W / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, W);
  return v;
}

template <int W>
__device__ __forceinline__ double group_incl_scan(double v, int li) {
#pragma unroll
  for (int o = 1; o < W; o <<= 1) {
    const double y = __shfl_up(v, o, W);
    if (li >= o) v += y;
  }
  return v;
}

// Shift a double right by S lanes inside each row of 16 lanes (DPP
// row_shr); lanes below S read 0.
template <int S>
__device__ __forceinline__ double row_shr(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x110 + S, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x110 + S, 0xF, 0xF, true);
  return __hiloint2double(hi, lo);
}

// Inclusive prefix sum over each row of 16 lanes.
__device__ __forceinline__ double row_incl_scan(double v) {
  v += row_shr<1>(v);
  v += row_shr<2>(v);
  v += row_shr<4>(v);
  v += row_shr<8>(v);
  return v;
}

// A double from another lane by a DPP control, in the rows of row_mask only
// (the other rows read 0).
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_rows_f64(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWS, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWS, 0xF, false);
  return __hiloint2double(hi, lo);
}

// Inclusive prefix sum over the 64 lanes of a wave: a scan per row, then
// row 0's total added to row 1 and row 2's to row 3 (row_bcast:15), then the
// total of rows 0 and 1 added to rows 2 and 3 (row_bcast:31).
__device__ __forceinline__ double wave_incl_scan(double v) {
  v = row_incl_scan(v);
  v += dpp_rows_f64<0x142, 0xA>(v);
  v += dpp_rows_f64<0x143, 0xC>(v);
  return v;
}

// Inclusive prefix sum of whole numbers over each row of 16 lanes.
template <int S>
__device__ __forceinline__ unsigned long long row_shr_u64(unsigned long long v) {
  const uint32_t lo = uint32_t(__builtin_amdgcn_update_dpp(0, int(uint32_t(v)), 0x110 + S, 0xF, 0xF, true));
  const uint32_t hi = uint32_t(__builtin_amdgcn_update_dpp(0, int(uint32_t(v >> 32)), 0x110 + S, 0xF, 0xF, true));
  return (unsigned long long)hi << 32 | lo;
}
__device__ __forceinline__ unsigned long long row_incl_scan_u64(unsigned long long v) {
  v += row_shr_u64<1>(v);
  v += row_shr_u64<2>(v);
  v += row_shr_u64<4>(v);
  v += row_shr_u64<8>(v);
  return v;
}

// A double from lane l (uniform) to every lane.
__device__ __forceinline__ double readlane_f64(double v, int l) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l), __builtin_amdgcn_readlane(__double2loint(v), l));
}

constexpr int kTop = 4;  // top values of W^[v] kept per word (a1..a4 of Eq. 9, g <= 3)

struct TopN {
  double v[kTop];
  uint32_t k[kTop];
};

__device__ __forceinline__ bool better(double va, uint32_t ka, double vb, uint32_t kb) {
  return va > vb || (va == vb && ka < kb);
}

// Insert (v, k) into a list kept in order of `better` (value descending,
// lowest topic id first among equal values).
__device__ __forceinline__ void top_insert(TopN &t, double v, uint32_t k) {
  if (!better(v, k, t.v[kTop - 1], t.k[kTop - 1])) return;
  t.v[kTop - 1] = v;
  t.k[kTop - 1] = k;
#pragma unroll
  for (int q = kTop - 1; q > 0; --q) {
    if (better(t.v[q], t.k[q], t.v[q - 1], t.k[q - 1])) {
      const double tv = t.v[q - 1];
      const uint32_t tk = t.k[q - 1];
      t.v[q - 1] = t.v[q];
      t.k[q - 1] = t.k[q];
      t.v[q] = tv;
      t.k[q] = tk;
    }
  }
}

// Block-wide sum of a double over 256 threads (fixed order).
__device__ double block_sum(double v, double *red) {
  v = group_sum<kWave>(v);
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  __syncthreads();
  if (lane == 0) red[wave] = v;
  __syncthreads();
  double s = 0.0;
  for (int q = 0; q < kBlock / kWave; ++q) s += red[q];
  __syncthreads();
  return s;
}

// A sum with the rounding errors of its additions beside it (Knuth's two-sum):
// h + l is off by about 2^-104 of the largest partial sum.
struct Sum2 {
  double h, l;
};
__device__ __forceinline__ Sum2 sum2_add(Sum2 a, Sum2 b) {
  const double s = a.h + b.h, bb = s - a.h;
  const double e = ((a.h - (s - bb)) + (b.h - bb)) + (a.l + b.l);
  const double h = s + e;
  return Sum2{h, e - (h - s)};
}
// One more value; h alone is the chain from value to value.
__device__ __forceinline__ void sum2_push(Sum2 &a, double b) {
  const double s = a.h + b, bb = s - a.h;
  a.l += (a.h - (s - bb)) + (b - bb);
  a.h = s;
}
// Over each group of G lanes, in every lane.
template <int G>
__device__ __forceinline__ Sum2 group_sum2(Sum2 a) {
#pragma unroll
  for (int o = G / 2; o > 0; o >>= 1) a = sum2_add(a, Sum2{__shfl_xor(a.h, o, kWave), __shfl_xor(a.l, o, kWave)});
  return a;
}
// Over the kBlock threads of a workgroup (fixed order), in every thread.
__device__ Sum2 block_sum2(Sum2 v, Sum2 *red) {
  v = group_sum2<kWave>(v);
  __syncthreads();
  if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x / kWave] = v;
  __syncthreads();
  Sum2 s = red[0];
  for (int q = 1; q < kBlock / kWave; ++q) s = sum2_add(s, red[q]);
  return s;
}

// Block-wide exclusive prefix of a uint32 over 256 threads; *total gets the sum.
__device__ uint32_t block_exclusive_u32(uint32_t v, uint32_t *red, uint32_t *total) {
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  uint32_t incl = v;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const uint32_t y = __shfl_up(incl, o, kWave);
    if (lane >= o) incl += y;
  }
  __syncthreads();
  if (lane == kWave - 1) red[wave] = incl;
  __syncthreads();
  uint32_t off = 0, all = 0;
  for (int q = 0; q < kBlock / kWave; ++q) {
    if (q < wave) off += red[q];
    all += red[q];
  }
  *total = all;
  return off + incl - v;
}

// First index in [0, nnz) whose packed topic is >= k.
__device__ __forceinline__ uint32_t row_lower_bound(const uint32_t *__restrict__ row, uint32_t nnz, uint32_t k) {
  uint32_t lo = 0, hi = nnz;
  while (lo < hi) {
    const uint32_t mid = (lo + hi) >> 1;
    if ((row[mid] >> 16) < k) lo = mid + 1;
    else hi = mid;
  }
  return lo;
}

// ------------------------------------------------------------ kernels ----

__device__ __forceinline__ uint16_t initial_topic(uint64_t seed, uint32_t i, int32_t K) {
  const uint4 x = philox4x32_10(make_uint4(i, 0u, 0u, 1u), uint32_t(seed), uint32_t(seed >> 32));
  return uint16_t((uint64_t(x.x) * uint64_t(uint32_t(K))) >> 32);
}

__global__ void k_init_topics(const uint2 *__restrict__ wt_kr, uint16_t *__restrict__ z_w, int64_t n, int32_t K,
                              uint64_t seed) {
  for (int64_t j = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; j < n; j += int64_t(gridDim.x) * blockDim.x)
    z_w[j] = initial_topic(seed, wt_kr[j].x, K);
}

// The skip bitmaps start every iteration clear, and so does this
// iteration's skip count (the other parity's count, the previous
// iteration's, stays for the choice of bitmap).
__global__ void k_clear_skips(uint32_t *__restrict__ bits, uint32_t *__restrict__ doc_bits, int64_t n, int64_t n_doc,
                              unsigned long long *__restrict__ hist, uint32_t t, int reset_count) {
  const int64_t i0 = int64_t(blockIdx.x) * blockDim.x + threadIdx.x, step = int64_t(gridDim.x) * blockDim.x;
  for (int64_t q = i0; q < n; q += step) bits[q] = 0u;
  if (doc_bits)
    for (int64_t q = i0; q < n_doc; q += step) doc_bits[q] = 0u;
  if (i0 == 0 && reset_count) hist[t & 1u] = 0ull;
}

__global__ void k_reset_counters(uint32_t *__restrict__ counters) {
  for (int i = int(threadIdx.x); i < kCounters; i += int(blockDim.x)) counters[i] = 0u;
}

// Whether iteration t carries its skip decisions in the document-ordered
// bitmap: coalesced writes in the doc pass and one dependent read per token
// in the sampler, against one scattered write per skipped token for the
// word-ordered bitmap.  By default it does once the previous iteration
// skipped more than a fifth of the tokens, where the scattered writes cost
// more than the reads.
__device__ __forceinline__ bool doc_marks(const DevState &d, const Params &p, uint32_t t) {
  if (!p.doc_marks_ok || p.skip_marks == 1) return false;
  if (p.skip_marks == 2) return true;
  return t > 0u && 5ull * d.skip_hist[(t + 1u) & 1u] > uint64_t(p.n_all);
}

// Whether steps 2-3 run in iteration t.  They only save work: a token they
// skip costs the sampler a bit test instead of its D row, so they pay once
// enough tokens skip (the doc pass costs about as much as the sampler work of
// a tenth of the tokens).  By default they run in every kProbeEvery-th
// iteration, which measures the skip rate, and in every iteration after one
// that skipped at least an eighth of the tokens; a token left unmarked is
// drawn in full, so the draws are the same either way.
constexpr uint32_t kProbeEvery = 8;
__device__ __forceinline__ bool skip_test_runs(const DevState &d, const Params &p, uint32_t t) {
  if (p.no_skip) return false;
  if (p.always_skip_test || t % kProbeEvery == 0u) return true;
  return 8ull * d.skip_hist[(t + 1u) & 1u] >= uint64_t(p.n_all);
}

__global__ void k_begin(const uint32_t *__restrict__ T, double *__restrict__ den, double *__restrict__ bden, int32_t K,
                        double beta, double vbeta, uint32_t *__restrict__ counters,
                        unsigned long long *__restrict__ stats) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k < K) {
    const double dk = double(T[k]) + vbeta;
    den[k] = dk;
    bden[k] = what(0u, beta, dk);  // W^[v][k] of every topic that word v does not hold
  }
  if (blockIdx.x == 0) {
    for (int i = int(threadIdx.x); i < kCounters; i += int(blockDim.x)) counters[i] = 0u;
    if (stats && threadIdx.x < kStatsPerIter) stats[threadIdx.x] = 0ull;
  }
}

// Step 1 of Sec. 3.2 and the per-word Q' of Sec. 2.2 (built once per word).
struct WordTop {
  uint32_t k1, k2, k3;
  double a1, a2, a3, a4;
};

__device__ __forceinline__ WordTop word_top_of(const TopN &t) {
  WordTop top;
  top.k1 = t.k[0];
  top.k2 = t.k[1];
  top.k3 = t.k[2];
  top.a1 = t.v[0];
  top.a2 = t.v[1];
  top.a3 = t.v[2] > 0.0 ? t.v[2] : 0.0;
  top.a4 = t.v[3] > 0.0 ? t.v[3] : 0.0;
  return top;
}

// The sampler's and the skip test's per-word records.  In two-branch mode
// (Sec. 2.2) the max-topic branch is empty (a1 = 0, K1 = K, a topic no row
// holds with a count) and Q' is the full Q.
__device__ void write_word_records(const DevState &d, const Params &p, int r, const WordTop &top, double q, double sw) {
  const int K = p.K;
  const uint32_t K3 = K >= 3 ? top.k3 : 0xFFFFFFFFu;
  WordRec rec;
  rec.a1 = p.two_branch ? 0.0 : top.a1;
  rec.a2 = top.a2;
  rec.a3 = K >= 3 ? top.a3 : 0.0;
  rec.qp = q;
  rec.sumw = sw;
  rec.k1 = p.two_branch ? uint32_t(K) : top.k1;
  rec.k2 = top.k2;
  d.wrec[r] = rec;
  SkipRec sr;
  sr.k12 = top.k1 | (top.k2 << 16);
  sr.k3 = K3;
  sr.a1 = float(top.a1);
  sr.a2 = float(top.a2);
  sr.a3 = float(K >= 3 ? top.a3 : 0.0);
  sr.a4 = float(K >= 4 ? top.a4 : 0.0);
  sr.qp = float(q);
  sr.pad = 0u;
  d.wskip[r] = sr;
}

// The sum over all topics of beta/den[k] (one workgroup, a fixed order) with
// its rounding error, for the sparse words' sums (RowSums).
__device__ __forceinline__ void beta_sum_all(const DevState &d, int K) {
  __shared__ Sum2 red[kBlock / kWave];
  Sum2 s{0.0, 0.0};
#pragma unroll 4
  for (int k = int(threadIdx.x); k < K; k += kBlock) sum2_push(s, d.bden[k]);
  s = block_sum2(s, red);
  if (threadIdx.x == 0) {
    d.beta_sum[0] = s.h;
    d.beta_sum[1] = s.l;
  }
}
// K from 4,096 on (below, k_topic_list's last workgroup).
__global__ __launch_bounds__(kBlock) void k_beta_sum(DevState d, Params p) { beta_sum_all(d, p.K); }

// Q' and the sum of W^[v] from `others`, the sum of W^[v] over every topic but
// K1.  It comes with its rounding errors (Sum2), so that the numbers are the
// exact sums rounded once: the same bits from a dense row, topic by topic, and
// from a sparse one (RowSums), and so the same draws.
__device__ __forceinline__ void write_word_sums(const DevState &d, const Params &p, int r, const WordTop &top, Sum2 others) {
  const double sw = sum2_add(others, Sum2{top.a1, 0.0}).h;
  write_word_records(d, p, r, top, p.alpha * (p.two_branch ? sw : others.h), sw);
}

// A sparse word's sums from its row, one lane's entries: the sum of W^ over
// every topic but K1 is the sum of beta/den[k] over all topics, less
// beta/den[k] of the row's topics, plus W^ of its entries other than K1.
// W^[v][K1] is never in it: taken off a plain sum, a K1 that holds nearly all
// of it would leave Q' with the rounding errors of the whole (up to 7e-9 of Q'
// for words of one topic at beta = 1e-9, K = 1,000).
struct RowSums {
  Sum2 rest{0.0, 0.0};    // W^ of the entries but the largest (lowest topic on ties), less their beta/den[k]
  double best = 0.0;      // W^ of the largest
  uint32_t best_k = 0xFFFFFFFFu;
  __device__ __forceinline__ void topic(double w, uint32_t k) {
    const bool b = better(w, k, best, best_k);
    sum2_push(rest, b ? best : w);
    best = b ? w : best;
    best_k = b ? k : best_k;
  }
  __device__ __forceinline__ void entry(double w, double bden, uint32_t k) {
    topic(w, k);
    sum2_push(rest, -bden);
  }
};
// The word's records, from the RowSums of its group of G lanes, K1 among them
// or outside the row; lane `leader` writes.  gmask: the group's lanes.
template <int G>
__device__ __forceinline__ void write_sparse_records(const DevState &d, const Params &p, int r, const TopN &t,
                                                     const RowSums &rs, unsigned long long gmask, bool leader) {
  const WordTop top = word_top_of(t);
  const bool mine = rs.best_k == top.k1;
  const bool in_row = (__ballot(mine) & gmask) != 0ull;
  Sum2 s = rs.rest;
  sum2_push(s, mine ? 0.0 : rs.best);
  s = sum2_add(group_sum2<G>(s), Sum2{d.beta_sum[0], d.beta_sum[1]});
  s = sum2_add(s, Sum2{in_row ? 0.0 : -top.a1, 0.0});
  if (leader) write_word_sums(d, p, r, top, s);
}

// Step 1 (Sec. 3.2) and Q' (Sec. 2.2), one wave per word, four words per
// workgroup, no workgroup barriers.  Lane l takes topics l, l + 64, ...: its top values, then a merge
// across the wave by exchanges at distances 32 down to 1 (the top set is
// unique under `better`, so every lane ends with the same list), then the sum
// of W^[v] over the other topics (write_word_sums).  Without
// p.sparse_pre a sparse row is spread into the wave's table of K counts first.
// With it (use_topic_list) a sparse word's W^ is beta/den[k] outside
// its row: its top values come from the row and from the first topics
// outside the row in the list of all topics by ascending T (descending
// beta/den[k], lowest id first on ties), 64 candidates of the list at a time;
// its sums from the sum of beta/den[k] over all topics and the row (RowSums).
// Should the list run out, every topic is scanned.  The words from
// p.small_begin on are then k_word_pre_small's.
__device__ __forceinline__ void wave_top_merge(TopN &t) {
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) {
    double pv[kTop];
    uint32_t pk[kTop];
#pragma unroll
    for (int q = 0; q < kTop; ++q) {
      pv[q] = __shfl_xor(t.v[q], o, kWave);
      pk[q] = uint32_t(__shfl_xor(int(t.k[q]), o, kWave));
    }
#pragma unroll
    for (int q = 0; q < kTop; ++q) top_insert(t, pv[q], pk[q]);
  }
}
__global__ __launch_bounds__(kBlock) void k_word_pre_wave(DevState d, Params p) {
  extern __shared__ uint16_t wtab[];  // without p.sparse_pre: [kBlock / kWave][(K + 1) & ~1]
  const int K = p.K, lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int r = blockIdx.x * (kBlock / kWave) + wave;
  if (r >= (p.sparse_pre ? p.small_begin : p.n_present)) return;  // a whole wave; nothing below waits on the workgroup
  const bool dense = r < p.n_dense;
  const int32_t *wrow = dense ? d.w_dense + size_t(r) * size_t(K) : nullptr;
  const uint32_t *ents = nullptr;
  uint32_t nnz = 0;
  if (!dense) {
    const int s = r - p.n_dense;
    ents = d.ws_ent + d.ws_cap[s];
    nnz = d.ws_nnz[s];
  }
  TopN t;
  auto reset = [&]() {
    for (int q = 0; q < kTop; ++q) {
      t.v[q] = -1.0;
      t.k[q] = 0xFFFFFFFFu;
    }
  };
  reset();
  if (!dense && p.sparse_pre) {
    RowSums rs;
    for (uint32_t q = uint32_t(lane); q < nnz; q += kWave) {
      const uint32_t ent = ents[q], k = ent >> 16;
      const double w = what(ent & 0xFFFFu, p.beta, d.den[k]);
      top_insert(t, w, k);
      rs.entry(w, d.bden[k], k);
    }
    const uint32_t want = uint32_t(min(kTop, K - int(nnz)));
    uint32_t found = 0;
    for (int i0 = 0; i0 < p.top_list && found < want; i0 += kWave) {
      const int i = i0 + lane;
      bool cand = false;
      uint32_t k = 0;
      if (i < p.top_list) {
        k = d.topic_order[i];
        const uint32_t lb = row_lower_bound(ents, nnz, k);
        cand = !(lb < nnz && (ents[lb] >> 16) == k);
      }
      const unsigned long long m = __ballot(cand);
      const uint32_t rank = __builtin_amdgcn_mbcnt_hi(uint32_t(m >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(m), 0u));
      if (cand && rank < want - found) top_insert(t, d.bden[k], k);
      found += min(uint32_t(__popcll(m)), want - found);
    }
    wave_top_merge(t);
    if (found >= want) {
      write_sparse_records<kWave>(d, p, r, t, rs, ~0ull, lane == 0);
      return;
    }
    reset();  // the list ran out: every topic below
  }
  const bool tab = !dense && !p.sparse_pre;
  uint16_t *ct = wtab + size_t(wave) * size_t((K + 1) & ~1);
  if (tab) {
    for (int k = lane; k < K; k += kWave) ct[k] = 0;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");  // a wave's LDS accesses run in order
    for (uint32_t q = uint32_t(lane); q < nnz; q += kWave) {
      const uint32_t ent = ents[q];
      ct[ent >> 16] = uint16_t(ent & 0xFFFFu);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  // counts: the dense row, the table, or (a large-K sparse row whose topic
  // list ran out) a search of the row
  auto count_of = [&](int k) -> uint32_t {
    if (dense) return uint32_t(wrow[k]);
    if (tab) return uint32_t(ct[k]);
    const uint32_t lb = row_lower_bound(ents, nnz, uint32_t(k));
    return lb < nnz && (ents[lb] >> 16) == uint32_t(k) ? (ents[lb] & 0xFFFFu) : 0u;
  };
  // kPreAhead topics per lane at a time, their loads issued together (a
  // dense row at K = 32,768 is 512 topics per lane)
  constexpr int kPreAhead = 8;
  auto batch = [&](int k0, double (&w)[kPreAhead]) {
    uint32_t c[kPreAhead];
    double dn[kPreAhead];
#pragma unroll
    for (int u = 0; u < kPreAhead; ++u) {
      const int k = min(k0 + u * kWave, K - 1);
      c[u] = count_of(k);
      dn[u] = d.den[k];
    }
#pragma unroll
    for (int u = 0; u < kPreAhead; ++u) w[u] = what(c[u], p.beta, dn[u]);
  };
  // one pass: the sum of all but the lane's largest W^, which is K1's or
  // belongs to the sum as well (a second pass over the row for the sums made
  // the precompute 0.31 ms instead of 0.28 at K = 32,768)
  RowSums rs;
  for (int k0 = lane; k0 < K; k0 += kPreAhead * kWave) {
    double w[kPreAhead];
    batch(k0, w);
#pragma unroll
    for (int u = 0; u < kPreAhead; ++u) {
      const uint32_t k = uint32_t(k0 + u * kWave);
      if (k < uint32_t(K)) {
        top_insert(t, w[u], k);
        rs.topic(w[u], k);
      }
    }
  }
  wave_top_merge(t);
  const WordTop top = word_top_of(t);
  sum2_push(rs.rest, rs.best_k == top.k1 ? 0.0 : rs.best);
  const Sum2 others = group_sum2<kWave>(rs.rest);
  if (lane == 0) write_word_sums(d, p, r, top, others);
}

// The topic list (the p.top_list topics of least T, ascending, lowest id first
// on ties) and the sum of beta/den[k], for K below 4,096: a topic's place is
// the number of topics before it, counted by four lanes over T in LDS (6 us
// at K = 1,000; the radix sort that large K uses takes five launches).  The
// last workgroup sums beta/den[k].
constexpr int kListTopics = kBlock / 4;  // topics per workgroup
__global__ __launch_bounds__(kBlock) void k_topic_list(DevState d, Params p) {
  extern __shared__ uint32_t ldsu[];  // [K rounded up to 4]
  const int K = p.K, tid = threadIdx.x;
  if (int(blockIdx.x) * kListTopics >= K) {
    beta_sum_all(d, K);
    return;
  }
  const int K4 = (K + 3) & ~3;
  for (int k = tid; k < K4; k += kBlock) ldsu[k] = k < K ? d.T[k] : 0xFFFFFFFFu;  // the padding is after every topic
  __syncthreads();
  const uint32_t k = blockIdx.x * uint32_t(kListTopics) + uint32_t(tid / 4);
  if (k >= uint32_t(K)) return;
  const uint32_t t = ldsu[k];
  uint32_t before = 0;
  const uint4 *t4 = reinterpret_cast<const uint4 *>(ldsu);
  for (uint32_t q = uint32_t(tid & 3); q < uint32_t(K4 / 4); q += 4u) {
    const uint4 v = t4[q];
    const uint32_t j = 4u * q;
    before += uint32_t(v.x < t || (v.x == t && j < k)) + uint32_t(v.y < t || (v.y == t && j + 1u < k)) +
              uint32_t(v.z < t || (v.z == t && j + 2u < k)) + uint32_t(v.w < t || (v.w == t && j + 3u < k));
  }
  before += uint32_t(__shfl_xor(int(before), 1, 4));
  before += uint32_t(__shfl_xor(int(before), 2, 4));
  if ((tid & 3) == 0 && before < uint32_t(p.top_list)) d.topic_order[before] = k;
}

// The per-word records of the small sparse words (at most kSmallWord tokens,
// the words from p.small_begin on) from their row and the topic list, as
// k_word_pre_wave makes them, by 16 lanes per word.  A whole wave per word
// spent most of its instructions on merging 64 lanes' top lists: a million
// words took 2.1 ms by tables of K = 1,000 counts.  A row has
// at most 64 entries, so the list (512 topics, or all) holds enough topics
// outside it.
__global__ __launch_bounds__(kBlock) void k_word_pre_small(DevState d, Params p) {
  __shared__ uint16_t s_topic[kBlock / kGroup][kSmallWord];
  const int K = p.K, li = threadIdx.x % kGroup, g = threadIdx.x / kGroup;
  const int grp = (threadIdx.x & (kWave - 1)) / kGroup;  // of the wave
  const int word = p.small_begin + int(blockIdx.x) * (kBlock / kGroup) + g;
  const int r = min(word, p.n_present - 1), s = r - p.n_dense;
  const uint32_t nnz = d.ws_nnz[s];
  const uint32_t *ents = d.ws_ent + d.ws_cap[s];
  TopN t;
#pragma unroll
  for (int q = 0; q < kTop; ++q) {
    t.v[q] = -1.0;
    t.k[q] = 0xFFFFFFFFu;
  }
  RowSums rs;
  uint32_t ent[kSmallWord / kGroup];
#pragma unroll
  for (int u = 0; u < int(kSmallWord) / kGroup; ++u) {
    const uint32_t q = uint32_t(li + u * kGroup);
    ent[u] = q < nnz ? ents[q] : 0u;
  }
#pragma unroll
  for (int u = 0; u < int(kSmallWord) / kGroup; ++u) {
    const uint32_t q = uint32_t(li + u * kGroup);
    if (q < nnz) {
      const uint32_t k = ent[u] >> 16;
      const double w = what(ent[u] & 0xFFFFu, p.beta, d.den[k]);
      top_insert(t, w, k);
      rs.entry(w, d.bden[k], k);
      s_topic[g][q] = uint16_t(k);
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // a wave's LDS accesses run in order
  const uint32_t want = uint32_t(min(kTop, K - int(nnz)));
  uint32_t found = 0;
  for (int i0 = 0; i0 < p.top_list && __ballot(found < want) != 0ull; i0 += kGroup) {
    const int i = i0 + li;
    bool cand = false;
    uint32_t k = 0;
    if (i < p.top_list && found < want) {
      k = d.topic_order[i];
      uint32_t lo = 0, hi = nnz;  // first entry whose topic is >= k
      while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if (s_topic[g][mid] < k) lo = mid + 1;
        else hi = mid;
      }
      cand = !(lo < nnz && s_topic[g][lo] == k);
    }
    const uint32_t m = uint32_t(__ballot(cand) >> (grp * kGroup)) & kGroupMask;
    const uint32_t rank = uint32_t(__popc(m & ((1u << li) - 1u)));
    if (cand && rank < want - found) top_insert(t, d.bden[k], k);
    found += min(uint32_t(__popc(m)), want - found);
  }
#pragma unroll
  for (int o = kGroup / 2; o > 0; o >>= 1) {
    double pv[kTop];
    uint32_t pk[kTop];
#pragma unroll
    for (int q = 0; q < kTop; ++q) {
      pv[q] = __shfl_xor(t.v[q], o, kWave);
      pk[q] = uint32_t(__shfl_xor(int(t.k[q]), o, kWave));
    }
#pragma unroll
    for (int q = 0; q < kTop; ++q) top_insert(t, pv[q], pk[q]);
  }
  write_sparse_records<kGroup>(d, p, r, t, rs, (unsigned long long)(kGroupMask) << (grp * kGroup),
                               li == 0 && word < p.n_present);
}

// Steps 2 and 3: per document, C1 = D[d][K1], C2 = D[d][K2], u, M, S_est and
// the skip test (Eq. 7 and 9).  One wave per document; documents are handed
// out in batches through an atomic counter.  The document's D row is spread
// into a per-wave topic -> count table in LDS, so each token's C1 and C2 are
// two LDS reads; the table is cleared again from the row afterwards.

// Next batch [d0, d1) of documents for a wave of the D rebuild.  The
// documents are split into kXcds ranges of equal token counts; workgroups are
// dealt to the XCDs in turn, so blockIdx.x % kXcds names the wave's XCD, and
// a wave takes batches from its own XCD's range first, then from the others
// in turn.  Each XCD's L2 then sees a compact window of documents, and the
// word-ordered topic slots that window gathers are fetched by one XCD
// instead of all of them.
__device__ __forceinline__ bool next_docs(uint32_t *__restrict__ cnt, const Params &p, int &part, int lane,
                                          uint32_t &d0, uint32_t &d1) {
  const int x = int(blockIdx.x % kXcds);
  while (part < kXcds) {
    const int r = (x + part) % kXcds;
    const uint32_t b0 = p.xcd_doc[r], e = p.xcd_doc[r + 1];
    uint32_t *c = cnt + r * kLine;
    uint32_t o = 0;
    // another XCD's range is looked at before it is counted down (the counter
    // only grows, so an old value costs at most a wasted atomic)
    if (lane == 0 && (part == 0 || __hip_atomic_load(c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < e - b0))
      o = atomicAdd(c, p.rebuild_batch);
    else if (lane == 0)
      o = e - b0;
    o = __shfl(o, 0);
    if (o < e - b0) {
      d0 = b0 + o;
      d1 = min(d0 + p.rebuild_batch, e);
      return true;
    }
    ++part;
  }
  return false;
}

// The fields of a skip record that the test needs at g <= 2 (the first 20
// bytes of the record: one 16-byte and one 4-byte load).
struct SkipHead {
  uint32_t k12;
  float a1, a2, a3, qp;
};
__device__ __forceinline__ SkipHead skip_head(const SkipRec *__restrict__ r) {
  return SkipHead{r->k12, r->a1, r->a2, r->a3, r->qp};
}

constexpr int kDocAhead = 2;  // chunks of 64 tokens per document loaded one document ahead

// Documents longer than this are walked by a whole workgroup in the doc pass
// and the D rebuild (the skew-aware mapping of Sec. 5.1: heavy units to
// workgroups, light ones to waves); the per-wave kernels skip them.
constexpr uint32_t kHeavyDoc = kHeavyDocTokens;

// Step 3 for token pp of a document of length len, in single precision with a
// relative margin of 2^-15, far above the fp32 rounding of these few
// operations (a few 2^-24): a token is skipped only if u*(M + S_est + Q') < M
// holds exactly, so its draw is K1 (S' <= S_est, Eq. 8-9).  cmap is the
// document's topic -> count table.
template <bool KeyId>
__device__ __forceinline__ bool skip_test(const DevState &d, const Params &p, uint32_t t, const uint16_t *cmap,
                                          uint32_t pp, uint32_t len, const SkipHead &h, uint32_t v) {
  const uint32_t K1 = h.k12 & 0xFFFFu, K2 = h.k12 >> 16;
  const uint32_t C1 = cmap[K1], C2 = cmap[K2];
  const uint32_t key = KeyId ? p.key_base + pp : d.dt_key[pp];
  const float u = float(uniform_draw(p.seed, t, key));
  const float Mm = h.a1 * (float(C1) + p.alpha_f);
  float Sest;
  if (p.g == 1) {
    Sest = h.a2 * float(len - C1);
  } else if (p.g == 2) {
    Sest = h.a2 * float(C2) + h.a3 * float(len - C1 - C2);
  } else {
    const SkipRec &r = d.wskip[v];
    const uint32_t C3 = r.k3 < uint32_t(p.K) ? uint32_t(cmap[r.k3]) : 0u;
    Sest = h.a2 * float(C2) + h.a3 * float(C3) + r.a4 * float(len - C1 - C2 - C3);
  }
  return !p.no_skip && (u * ((Mm + Sest) + h.qp) < Mm * (1.0f - 0x1p-15f));
}

// A skipped token's decision goes to the sampler either as a bit at its
// word-order slot (one scattered write per skipped token) or, in the
// document-ordered bitmap, as a bit at its document position: a chunk's 64
// bits (lanes = positions p0 + lane) from a ballot, in at most three words,
// whose neighbours other waves may set too.
__device__ __forceinline__ void mark_slot(const DevState &d, uint32_t slot) {
  atomicOr(&d.skip_bits[slot >> 5], 1u << (slot & 31u));
}
__device__ __forceinline__ void mark_chunk(const DevState &d, unsigned long long m, uint32_t p0, int lane) {
  if (m == 0ull) return;
  const uint32_t sh = p0 & 31u;
  const uint32_t v0 = uint32_t(m << sh);
  const uint32_t v1 = sh ? uint32_t(m >> (32u - sh)) : uint32_t(m >> 32);
  const uint32_t v2 = sh ? uint32_t(m >> (64u - sh)) : 0u;
  const uint32_t v = lane == 0 ? v0 : lane == 1 ? v1 : v2;
  if (lane < 3 && v != 0u) atomicOr(&d.skip_doc[(p0 >> 5) + uint32_t(lane)], v);
}

template <bool KeyId>
__device__ void heavy_doc_pass(const DevState &d, const Params &p, uint32_t t, uint16_t *__restrict__ cmap,
                               bool by_doc, unsigned long long &nskip);

// Steps 2-3 per document (Sec. 3.3): the D row spread into a per-wave
// topic -> count table in LDS, then for every token C1 and C2 by lookup, u,
// M, S_est and the skip test.  A skipped token's bit is set in the
// word-ordered skip bitmap (one scattered bit at its word-order slot) or, in
// the iterations doc_marks chooses, in the document-ordered one (coalesced
// bits at its document position); the sampler writes K1 into its slot with
// the rest of its batch.  KeyId: the input is sorted by document, so a
// token's key (its input index) is its document-order position.
template <bool KeyId>
__global__ __launch_bounds__(kBlock) void k_doc_pass(DevState d, Params p, uint32_t t,
                                                     unsigned long long *__restrict__ stats) {
  extern __shared__ uint16_t cmap_all[];
  if (!skip_test_runs(d, p, t)) {  // uniform over the grid
    if (threadIdx.x % kWave == 0)
      d.wave_stats[size_t(WV_SKIP3) * kWaveSlots + blockIdx.x * uint32_t(p.doc_waves) + threadIdx.x / kWave] = 0ull;
    return;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) stats[ST_TEST_RAN] = 1ull;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int K = p.K;
  uint16_t *cmap = cmap_all + size_t(wave) * size_t(K);
  for (int k = lane; k < K; k += kWave) cmap[k] = 0;
  unsigned long long nskip = 0;
  const bool by_doc = doc_marks(d, p, t);
  // the heavy documents first, each by the whole workgroup (wave 0's table shared)
  if (p.n_heavy) heavy_doc_pass<KeyId>(d, p, t, cmap_all, by_doc, nskip);
  const uint32_t M = uint32_t(p.M);
  const uint32_t last = uint32_t(p.n - 1);
  auto test = [&](uint32_t pp, uint32_t len, const SkipHead &h, uint32_t v) -> bool {
    return skip_test<KeyId>(d, p, t, cmap, pp, len, h, v);
  };
  for (;;) {
    // batches i, i + kDocStripes, ... from the workgroup's stripe's counter
    const uint32_t stripe = blockIdx.x % uint32_t(kDocStripes);
    uint32_t o = 0;
    if (lane == 0) o = atomicAdd(&d.counters[CNT_DOCPASS + stripe * uint32_t(kLine)], 1u);
    o = __builtin_amdgcn_readfirstlane(__shfl(o, 0));
    const uint64_t first = (uint64_t(o) * uint32_t(kDocStripes) + stripe) * p.doc_batch;
    if (first >= M) break;
    const uint32_t d0 = uint32_t(first);
    const int nd = int(min(M, d0 + p.doc_batch) - d0);
    // the batch's document offsets and row offsets, one per lane
    const uint32_t offv = lane <= nd ? d.doc_off[d0 + uint32_t(lane)] : 0u;
    const uint32_t capv = lane < nd ? d.d_cap[d0 + uint32_t(lane)] : 0u;
    // Pipeline over the first kDocAhead*64 tokens and row slots of each
    // document: while document i is processed, the first row slots of
    // document i+1 (its header and entries), the skip records of the words
    // of document i+1 and the word ids of document i+2 are loaded.  Every
    // load is issued (indexes past the batch are clamped; lanes past a
    // document's end read word 0's record), so that the waits count a fixed
    // number of loads.
    auto rows_of = [&](int doc, uint32_t (&r)[kDocAhead]) {
      const uint32_t cap = __builtin_amdgcn_readlane(capv, doc);  // 0 past the batch; kRowPad covers the reach
#pragma unroll
      for (int c = 0; c < kDocAhead; ++c) r[c] = d.d_ent[cap + uint32_t(c * kWave + lane)];
    };
    auto words_of = [&](int doc, uint32_t (&w)[kDocAhead]) {
      const uint32_t bn = __builtin_amdgcn_readlane(offv, doc);
#pragma unroll
      for (int c = 0; c < kDocAhead; ++c) w[c] = d.dt_word[min(bn + uint32_t(c * kWave + lane), last)];
    };
    auto heads_of = [&](int doc, const uint32_t (&w)[kDocAhead], SkipHead (&h)[kDocAhead]) {
      const uint32_t bn = __builtin_amdgcn_readlane(offv, doc), en = __builtin_amdgcn_readlane(offv, doc + 1);
#pragma unroll
      for (int c = 0; c < kDocAhead; ++c) {
        const uint32_t pn = bn + uint32_t(c * kWave + lane);
        h[c] = skip_head(d.wskip + (pn < en ? w[c] : 0u));
      }
    };
    uint32_t rowA[kDocAhead], wA[kDocAhead], wB[kDocAhead];
    SkipHead hA[kDocAhead];
    rows_of(0, rowA);
    words_of(0, wA);
    words_of(1, wB);
    heads_of(0, wA, hA);
    for (int i = 0; i < nd; ++i) {
      const uint32_t b = __builtin_amdgcn_readlane(offv, i), e = __builtin_amdgcn_readlane(offv, i + 1);
      const uint32_t cap = __builtin_amdgcn_readlane(capv, i);
      const uint32_t len = e - b;
      uint32_t rowv[kDocAhead], wv[kDocAhead];
      SkipHead hv[kDocAhead];
#pragma unroll
      for (int c = 0; c < kDocAhead; ++c) {
        rowv[c] = rowA[c];
        hv[c] = hA[c];
        wv[c] = wA[c];
        wA[c] = wB[c];
      }
      rows_of(i + 1, rowA);
      words_of(i + 2, wB);
      heads_of(i + 1, wA, hA);
      if (len > kHeavyDoc) continue;  // a workgroup's document (heavy_doc_pass)
      const uint32_t *row = d.d_ent + cap + 1;  // entries; slot 0 is the header
      const uint32_t nnz = uint32_t(__builtin_amdgcn_readfirstlane(int(rowv[0]))) & 0xFFFFu;
      // spread the row into the topic -> count table
#pragma unroll
      for (int c = 0; c < kDocAhead; ++c) {
        const uint32_t q = uint32_t(c * kWave + lane);  // slot; entry q - 1
        if (q >= 1u && q <= nnz) cmap[rowv[c] >> 16] = uint16_t(rowv[c] & 0xFFFFu);
      }
      for (uint32_t q = uint32_t(kDocAhead * kWave - 1 + lane); q < nnz; q += kWave) {
        const uint32_t ent = row[q];
        cmap[ent >> 16] = uint16_t(ent & 0xFFFFu);
      }
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int c = 0; c < kDocAhead; ++c) {
        const uint32_t pp = b + uint32_t(c * kWave + lane);
        const bool skip = pp < e && test(pp, len, hv[c], wv[c]);
        nskip += skip ? 1ull : 0ull;
        if (by_doc) mark_chunk(d, __ballot(skip), b + uint32_t(c * kWave), lane);
        else if (skip) mark_slot(d, d.dt_wpos[pp]);
      }
      // the rest of a long document, two chunks per step
      for (uint32_t p0 = b + uint32_t(kDocAhead * kWave); p0 < e; p0 += 2u * kWave) {
        uint32_t v[2];
        SkipHead h[2];
#pragma unroll
        for (int c = 0; c < 2; ++c) v[c] = d.dt_word[min(p0 + uint32_t(c * kWave + lane), last)];
#pragma unroll
        for (int c = 0; c < 2; ++c) h[c] = skip_head(d.wskip + (p0 + uint32_t(c * kWave + lane) < e ? v[c] : 0u));
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          const uint32_t pp = p0 + uint32_t(c * kWave + lane);
          const bool skip = pp < e && test(pp, len, h[c], v[c]);
          nskip += skip ? 1ull : 0ull;
          if (by_doc) mark_chunk(d, __ballot(skip), p0 + uint32_t(c * kWave), lane);
          else if (skip) mark_slot(d, d.dt_wpos[pp]);
        }
      }
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int c = 0; c < kDocAhead; ++c) {
        const uint32_t q = uint32_t(c * kWave + lane);
        if (q >= 1u && q <= nnz) cmap[rowv[c] >> 16] = 0;
      }
      for (uint32_t q = uint32_t(kDocAhead * kWave - 1 + lane); q < nnz; q += kWave) cmap[row[q] >> 16] = 0;
      __builtin_amdgcn_wave_barrier();
    }
  }
  nskip = group_sum_u64<kWave>(nskip);
  if (lane == 0)
    d.wave_stats[size_t(WV_SKIP3) * kWaveSlots + blockIdx.x * uint32_t(p.doc_waves) + uint32_t(wave)] = nskip;
}

// Steps 2-3 for the heavy documents (longer than kHeavyDoc), one workgroup
// per document, taken from a list (d.heavy_docs) through one atomic counter
// before the workgroup's waves turn to the light documents: the D row spread
// into a topic -> count table shared by the workgroup (cmap, left clear),
// then each wave tests chunks of 64 consecutive tokens.
template <bool KeyId>
__device__ void heavy_doc_pass(const DevState &d, const Params &p, uint32_t t, uint16_t *__restrict__ cmap,
                               bool by_doc, unsigned long long &nskip) {
  __shared__ uint32_t s_next;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave, nthr = int(blockDim.x);
  for (;;) {
    __syncthreads();  // the table is clear, s_next is free
    if (tid == 0) s_next = atomicAdd(&d.counters[CNT_HEAVY_PASS], 1u);
    __syncthreads();
    const uint32_t h = s_next;
    if (h >= uint32_t(p.n_heavy)) break;
    const uint32_t dd = d.heavy_docs[h];
    const uint32_t b = d.doc_off[dd], e = d.doc_off[dd + 1], len = e - b;
    const uint32_t *row = d.d_ent + d.d_cap[dd];  // header, then the entries
    const uint32_t nnz = row[0] & 0xFFFFu;
    for (uint32_t q = uint32_t(tid); q < nnz; q += uint32_t(nthr)) {
      const uint32_t ent = row[1u + q];
      cmap[ent >> 16] = uint16_t(ent & 0xFFFFu);
    }
    __syncthreads();
    for (uint32_t p0 = b + uint32_t(wave * kWave); p0 < e; p0 += uint32_t(nthr)) {
      const uint32_t pp = p0 + uint32_t(lane);
      bool skip = false;
      if (pp < e) {
        const uint32_t v = d.dt_word[pp];
        skip = skip_test<KeyId>(d, p, t, cmap, pp, len, skip_head(d.wskip + v), v);
      }
      nskip += skip ? 1ull : 0ull;
      if (by_doc) mark_chunk(d, __ballot(skip), p0, lane);
      else if (skip) mark_slot(d, d.dt_wpos[pp]);
    }
    __syncthreads();
    for (uint32_t q = uint32_t(tid); q < nnz; q += uint32_t(nthr)) cmap[row[1u + q] >> 16] = 0;
  }
  __syncthreads();  // wave 0's table is clear again
}

// Steps 4-6 for the tokens of one region that step 3 left to draw; the W^ row of the word
// sits in LDS (Sec. 4.3, last paragraph) together with the Q' prefix over
// blocks of kGroup topics.
//
// Work split: a wave takes 64 consecutive word-ordered tokens.  Each lane
// loads its token's skip bit, key and D-row offset, and for a token left to
// draw its row header and u, staged in the wave's slice of LDS.  Those
// tokens are listed by row length and drawn in rounds by groups of 4, 8 or
// 16 lanes (draw_batch_small); rows over 512 slots by 16-lane groups in
// chunks (draw_long).  A group holds the row in registers (lane l a
// contiguous run, so lane partial sums are in ascending topic order), picks
// out C1 = D[d][K1], sums S', splits x between M, S' and Q', and records the
// selected run (S') or the remainder (Q'); one lane per token then finishes
// the draw (finish_draw).  The batch's topics, K1 for the skipped tokens,
// leave in one coalesced store.
static_assert(kGroup == 16, "the row scans use DPP rows of 16 lanes");
constexpr int kMaxRun = 8;                            // D entries per lane in registers
constexpr uint32_t kChunk = kGroup * kMaxRun;         // 128 entries per group per chunk

// One batch of 64 word-ordered tokens, staged in the wave's slice of LDS
// (entry q = lane q's token): D-row offset, row length, u, and the drawn topic.
struct BatchLds {
  uint32_t *off, *nnz;
  double *u;
  uint16_t *top;
  uint32_t *hand;  // kMaxRun slots per group: the selected lane's run
  uint8_t *list;   // the batch's lanes, sorted by row length, for the small-group draws
};

// The word of the current region: W^ row (with W^[K1] = 0) and Q' block
// prefix in LDS, and its per-word scalars.
struct WordState {
  const double *wh, *qb;
  int nb, K;
  int qhalf;  // half the padded block count of qb (0 for a single block): the binary search's first step
  uint32_t K1;
  double a1, qp, alpha;
  const double *qw;   // kQwStride per block: the partial sums before each of its kGroup topics, then its total (or null)
  const uint8_t *ql;  // per block: the offset of its last topic with a positive term (or its first)
};
constexpr int kQwStride = kGroup + 1;


// W^' of a packed D entry's topic (entry = topic << 16 | count) from the
// row in LDS: the address, topic * 8 + the row's LDS offset, is one
// v_mad_u32_u16 on the entry's high half (op_sel), read as an LDS pointer.
typedef const __attribute__((address_space(3))) double lds_f64;
__device__ __forceinline__ double wh_of(const double *__restrict__ wh, uint32_t e) {
  uint32_t a;
  asm("v_mad_u32_u16 %0, %1, 8, %2 op_sel:[1,0,0,0]"
      : "=v"(a)
      : "v"(e), "s"(uint32_t(reinterpret_cast<uintptr_t>(wh))));
  return *(lds_f64 *)(size_t)a;
}

// Load C entries per lane from `row` (lane li gets entries [li*C, li*C + C),
// topics ascending).  The row is padded to its length class with count-0
// entries of topic K, so all 16*C entries are in the row's slots.
template <int C>
__device__ __forceinline__ void load_run(const uint32_t *__restrict__ row, int li, uint32_t (&r)[C]) {
  const uint32_t q0 = uint32_t(li) * C;
#pragma unroll
  for (int i = 0; i < C; ++i) r[i] = row[q0 + i];
}

// This lane's S' terms in ascending topic order (W^[K1] = 0 in LDS).  The
// lane sums are fused multiply-adds: S' is a sum in another association than
// the sequential one anyway, so only draws within rounding distance of a
// segment boundary can depend on it.
template <int C>
__device__ __forceinline__ double run_sum(const uint32_t (&r)[C], const double *__restrict__ wh) {
  double s = 0.0;
#pragma unroll
  for (int i = 0; i < C; ++i) s = __builtin_fma(double(r[i] & 0xFFFFu), wh_of(wh, r[i]), s);
  return s;
}

// min(c, D[d][K1]) if this lane's run holds topic K1, else c unchanged or
// larger than 0xFFFF: an entry minus (K1 << 16) is its count when its topic
// is K1 and at least 2^16 (modulo 2^32) for any other topic, since topics
// (and the padding topic K) are below 2^16.
template <int C>
__device__ __forceinline__ uint32_t run_count_of(const uint32_t (&r)[C], uint32_t K1, uint32_t c) {
  const uint32_t key = K1 << 16;
#pragma unroll
  for (int i = 0; i < C; ++i) c = min(c, r[i] - key);
  return c;
}

// Sum of a uint32 over each row of 16 lanes, in every lane of the row.
__device__ __forceinline__ uint32_t row_sum_u32(uint32_t v) {
  v += uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x111, 0xF, 0xF, true));
  v += uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x112, 0xF, 0xF, true));
  v += uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x114, 0xF, 0xF, true));
  v += uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x118, 0xF, 0xF, true));
  return __shfl(v, kGroup - 1, kGroup);
}

// Sum of a uint32 over the wave (the total must fit in 32 bits), as a
// wave-uniform value.
__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t v) {
  v += uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x111, 0xF, 0xF, true));
  v += uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x112, 0xF, 0xF, true));
  v += uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x114, 0xF, 0xF, true));
  v += uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x118, 0xF, 0xF, true));
  return uint32_t(__builtin_amdgcn_readlane(int(v), 15)) + uint32_t(__builtin_amdgcn_readlane(int(v), 31)) +
         uint32_t(__builtin_amdgcn_readlane(int(v), 47)) + uint32_t(__builtin_amdgcn_readlane(int(v), 63));
}

// Lane of the row whose run holds x: the first lane with terms whose
// inclusive prefix passes x, else (rounding) the last lane with terms.
__device__ __forceinline__ int run_lane(double s, double incl, double base, double x, int grp) {
  const uint32_t hm = uint32_t(__ballot(s > 0.0 && x < base + incl) >> (grp * kGroup)) & kGroupMask;
  const uint32_t pm = uint32_t(__ballot(s > 0.0) >> (grp * kGroup)) & kGroupMask;
  return hm ? __ffs(hm) - 1 : (pm ? 31 - __clz(pm) : 0);
}

// Block b of the Q' prefix holding xq: the largest b in [0, nb) with
// qb[b] <= xq, found 16 candidates at a time.
__device__ __forceinline__ int q_block(double xq, const WordState &w, int grp, int li) {
  int lo = 0, span = w.nb;
  while (span > 1) {
    const int step = (span + kGroup - 1) / kGroup;
    const int off = li * step;
    const bool ok = off < span && w.qb[lo + off] <= xq;
    const uint32_t bm = uint32_t(__ballot(ok) >> (grp * kGroup)) & kGroupMask;
    const int best = bm ? 31 - __clz(bm) : 0;
    lo += best * step;
    span = min(step, span - best * step);
  }
  return lo;
}

// The last step of every draw: 16 candidate segments, one per lane (lane li
// holds topic k_li with width term_li >= 0, in canonical order after
// `start`); returns the topic of the first segment whose running sum passes
// x (the last positive one if rounding leaves x past them all).
__device__ __forceinline__ uint32_t pick_segment(uint32_t k, double term, double start, double x, int grp) {
  const double in2 = row_incl_scan(term);
  const uint32_t hm = uint32_t(__ballot(term > 0.0 && x < start + in2) >> (grp * kGroup)) & kGroupMask;
  const uint32_t pm = uint32_t(__ballot(term > 0.0) >> (grp * kGroup)) & kGroupMask;
  const int h = hm ? __ffs(hm) - 1 : (pm ? 31 - __clz(pm) : 0);
  return __shfl(k, h, kGroup);
}

// Draw the tokens of `mask` (rows longer than the small-group rounds take),
// four at a time, one per 16-lane group, walking each row in chunks of
// kChunk entries.  `foll` marks the later tokens of runs of one word in one
// document (same row; `starts` marks where runs begin): they share the row,
// M, S' and Q' with the run's first token (Sec. 3.3), so the group that draws
// the first one also draws them from the sums it holds, reading at most the
// one chunk that holds each x.  Every draw is the one the token would get on
// its own, bit for bit.
// Sum: no draw; bt.u of every token gets the sum of its row's terms.
template <bool Sum>
__device__ void draw_long(unsigned long long mask, unsigned long long foll, unsigned long long starts,
                          const BatchLds &bt, const WordState &w, const uint32_t *__restrict__ d_ent, int grp, int li,
                          uint32_t &after_s) {
  constexpr int R = kMaxRun;
  mask &= ~foll;  // the runs' first tokens
  while (mask) {
    // the four lowest tokens of the mask, one per group (wave-uniform bit
    // arithmetic; a group with none gets src = -1)
    const unsigned long long m1 = mask & (mask - 1ull), m2 = m1 & (m1 - 1ull), m3 = m2 & (m2 - 1ull);
    const int f0 = __ffsll((long long)mask) - 1, f1 = __ffsll((long long)m1) - 1;
    const int f2 = __ffsll((long long)m2) - 1, f3 = __ffsll((long long)m3) - 1;
    mask = m3 & (m3 - 1ull);
    const int src = grp == 0 ? f0 : grp == 1 ? f1 : grp == 2 ? f2 : f3;
    uint32_t n_m = 0;  // draws of this group in the max-topic branch
    if (src >= 0) {
    const uint32_t t_off = bt.off[src];
    const uint32_t t_nnz = bt.nnz[src];
    const uint32_t *row = d_ent + t_off;  // slot 0 is the row header
    const uint32_t pad = uint32_t(w.K) << 16;
    const uint32_t nch = (t_nnz + 1u + kChunk - 1) / kChunk;
    uint32_t r[R];
    double s = 0.0, incl = 0.0, S = 0.0;
    double tot = 0.0;  // lane c of the group (c < kGroup): the total of chunk c
    uint32_t c1 = 0xFFFFFFFFu;
    for (uint32_t ch = 0; ch < nch; ++ch) {
      load_run<R>(row + ch * kChunk, li, r);
      if (ch == 0u && li == 0) r[0] = pad;
      if (!Sum) c1 = run_count_of<R>(r, w.K1, c1);
      s = run_sum<R>(r, w.wh);
      incl = row_incl_scan(s);
      const double tch = __shfl(incl, kGroup - 1, kGroup);
      S += tch;
      tot = uint32_t(li) == ch ? tch : tot;
    }
    // the run's later tokens: lanes after src up to the next run start
    const unsigned long long after = ~((2ull << src) - 1ull);  // the lanes above src
    const unsigned long long nxt = starts & after;
    unsigned long long fl = foll & after & (nxt ? (nxt & (0ull - nxt)) - 1ull : ~0ull);
    if constexpr (Sum) {
      if (li == 0) bt.u[src] = S;
      for (; fl; fl &= fl - 1ull)
        if (li == 0) bt.u[__ffsll((long long)fl) - 1] = S;
    } else {
    // max-topic branch, Eq. 7: M = W^[v][K1] * (D[d][K1] + alpha)
    const double Mm = w.a1 * (double(row_sum_u32(c1 <= 0xFFFFu ? c1 : 0u)) + w.alpha);
    // with the totals kept in the lanes: lane c's chunk base
    // M + t_0 + ... + t_(c-1), added left to right as the walk over the
    // chunks adds them, and the base after the last chunk
    const bool kept = nch > 1 && nch <= uint32_t(kGroup);
    double mine = Mm, cb_end = Mm;
    if (kept) {
      for (uint32_t c = 0; c < nch; ++c) {
        mine = uint32_t(li) == c ? cb_end : mine;
        cb_end += __shfl(tot, int(c), kGroup);
      }
    }
    // the draw of one token of the row from x = u * Z
    auto draw_x = [&](double x) -> uint32_t {
      if (x < Mm) {
        n_m++;
        return w.K1;
      }
      // locate the chunk, then 16 candidate segments
      double cbase = Mm;
      bool in_s = false;
      if (kept) {
        // only the chunk that holds x is read again
        const uint32_t hm = uint32_t(__ballot(uint32_t(li) < nch && x < mine + tot) >> (grp * kGroup)) & kGroupMask;
        cbase = cb_end;
        if (hm) {
          const int cs = __ffs(hm) - 1;
          in_s = true;
          cbase = __shfl(mine, cs, kGroup);
          load_run<R>(row + uint32_t(cs) * kChunk, li, r);
          if (cs == 0 && li == 0) r[0] = pad;
          s = run_sum<R>(r, w.wh);
          incl = row_incl_scan(s);
        }
      } else {
        for (uint32_t ch = 0; ch < nch && !in_s; ++ch) {
          if (nch > 1) {
            load_run<R>(row + ch * kChunk, li, r);
            if (ch == 0u && li == 0) r[0] = pad;
            s = run_sum<R>(r, w.wh);
            incl = row_incl_scan(s);
          }
          const double total = __shfl(incl, kGroup - 1, kGroup);
          if (x < cbase + total) in_s = true;
          else cbase += total;
        }
      }
      uint32_t k;
      double term, start;
      if (in_s) {
        // S' run of one lane, moved across the group
        const int sel = run_lane(s, incl, cbase, x, grp);
        start = cbase + __shfl(incl - s, sel, kGroup);
        // lane li < R of the group takes entry li of the selected run
        uint32_t *hand = bt.hand + grp * kMaxRun;
        if (li == sel) {
#pragma unroll
          for (int i = 0; i < R; ++i) hand[i] = r[i];
        }
        const uint32_t own = li < R ? hand[li] : 0u;
        k = own >> 16;
        term = double(own & 0xFFFFu) * w.wh[k];
      } else {
        // Q' branch: boundaries (M + S') + Qcdf
        const double qstart = cbase;
        const double xq = x - qstart;
        if (!(xq < w.qb[w.nb])) {
          k = (w.K1 == uint32_t(w.K - 1)) ? uint32_t(w.K - 2) : uint32_t(w.K - 1);  // last positive segment
          term = 0.0;
          start = 0.0;
        } else {
          const int lo = q_block(xq, w, grp, li);
          k = uint32_t(lo * kGroup + li);
          term = int(k) < w.K ? w.alpha * w.wh[k] : 0.0;
          start = qstart + w.qb[lo];
        }
      }
      const bool fallback = !in_s && term == 0.0 && start == 0.0;
      const uint32_t picked = pick_segment(k, term, start, x, grp);
      return fallback ? k : picked;
    };
    const uint32_t topic = draw_x(bt.u[src] * ((Mm + S) + w.qp));
    if (li == 0) bt.top[src] = uint16_t(topic);
    while (fl) {
      const int f = __ffsll((long long)fl) - 1;
      fl &= fl - 1ull;
      const uint32_t tf = draw_x(bt.u[f] * ((Mm + S) + w.qp));
      if (li == 0) bt.top[f] = uint16_t(tf);
    }
    }
    }
    // outside the divergent part, so the count stays wave-uniform
    if (!Sum) after_s += wave_sum_u32(li == 0 ? n_m : 0u);
  }
}

// Entries of the sampler's W^' row in LDS: K + 1 (topic K is the padding of
// D rows) rounded up to whole blocks of kGroup topics, zeros past K.
__host__ __device__ inline int wh_entries(int K) { return (K + 1 + kGroup - 1) / kGroup * kGroup; }

// Blocks of the Q' prefix rounded up to a power of 2 (its binary search).
__host__ __device__ inline int q_blocks_padded(int nb) {
  int q = 1;
  while (q < nb) q *= 2;
  return q;
}

// ------------------------------------------------ small-group draws ----
// Rows of at most 512 slots are drawn by groups of G = 4 lanes (rows of up
// to 128 slots, 16 tokens per wave at a time), G = 8 lanes (up to 256 slots,
// 8 tokens at a time) or G = 16 lanes (up to 512 slots, 4 tokens), in chunks
// of G*kRun slots whose loads are all issued before the first is used.
// Group-wide sums and scans are DPP moves inside quads (quad_perm), half
// rows (row_half_mirror) and rows (row_mirror); the selected entry is found
// by a walk inside one lane.
constexpr int kRun = 8;
constexpr int kDppXor1 = 0xB1;         // quad_perm [1,0,3,2]
constexpr int kDppXor2 = 0x4E;         // quad_perm [2,3,0,1]
constexpr int kDppHalfMirror = 0x141;  // lane i <- lane 7-i inside each 8 lanes
constexpr int kDppMirror = 0x140;      // lane i <- lane 15-i inside each 16 lanes

template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t v) {
  return uint32_t(__builtin_amdgcn_update_dpp(0, int(v), CTRL, 0xF, 0xF, true));
}
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xF, 0xF, true);
  return __hiloint2double(hi, lo);
}

// Sum over a group of G (4, 8 or 16) aligned lanes; every lane gets the
// same bits (each step adds a pair in both orders, and IEEE addition
// commutes).
template <int G>
__device__ __forceinline__ double gsum(double v) {
  v += dpp_f64<kDppXor1>(v);
  v += dpp_f64<kDppXor2>(v);
  if (G >= 8) v += dpp_f64<kDppHalfMirror>(v);
  if (G >= 16) v += dpp_f64<kDppMirror>(v);
  return v;
}
template <int G>
__device__ __forceinline__ uint32_t gsum_u32(uint32_t v) {
  v += dpp_u32<kDppXor1>(v);
  v += dpp_u32<kDppXor2>(v);
  if (G >= 8) v += dpp_u32<kDppHalfMirror>(v);
  if (G >= 16) v += dpp_u32<kDppMirror>(v);
  return v;
}
template <int G>
__device__ __forceinline__ uint32_t gmin_u32(uint32_t v) {
  v = min(v, dpp_u32<kDppXor1>(v));
  v = min(v, dpp_u32<kDppXor2>(v));
  if (G >= 8) v = min(v, dpp_u32<kDppHalfMirror>(v));
  if (G >= 16) v = min(v, dpp_u32<kDppMirror>(v));
  return v;
}
template <int G>
__device__ __forceinline__ uint32_t gmax_u32(uint32_t v) {
  v = max(v, dpp_u32<kDppXor1>(v));
  v = max(v, dpp_u32<kDppXor2>(v));
  if (G >= 8) v = max(v, dpp_u32<kDppHalfMirror>(v));
  if (G >= 16) v = max(v, dpp_u32<kDppMirror>(v));
  return v;
}
// Inclusive prefix sum over a group of G lanes (li = lane in the group).
template <int G>
__device__ __forceinline__ double gscan(double v, int li) {
  { const double t = row_shr<1>(v); v += li >= 1 ? t : 0.0; }
  { const double t = row_shr<2>(v); v += li >= 2 ? t : 0.0; }
  if (G >= 8) { const double t = row_shr<4>(v); v += li >= 4 ? t : 0.0; }
  if (G >= 16) { const double t = row_shr<8>(v); v += li >= 8 ? t : 0.0; }
  return v;
}

// Segment of a group's CDF that holds x: the group's lanes carry terms s >= 0
// (in canonical order, lane by lane) whose inclusive scan is incl, starting at
// base.  Returns the first lane whose range passes x, or, when rounding puts x
// at or past the end, the last lane with a positive term.
template <int G>
__device__ __forceinline__ int pick_lane(double s, double incl, double base, double x, int li) {
  const uint32_t n = gsum_u32<G>(x >= base + incl ? 1u : 0u);
  if (n < uint32_t(G)) return int(n);
  return int(gmax_u32<G>(s > 0.0 ? uint32_t(li) : 0u));
}

// First of kRun packed entries whose running S' sum (fused multiply-adds from
// 0, as in run_sum) passes xs >= 0; the last entry with a positive term if
// rounding leaves xs at or past the lane's total.  Such an entry always has
// a positive term.
__device__ __forceinline__ uint32_t walk_run(const uint32_t (&r)[kRun], const double *__restrict__ wh, double xs) {
  double p = 0.0;
  uint32_t ent = r[0];
#pragma unroll
  for (int i = 0; i < kRun; ++i) {
    const bool open = p <= xs;
    p = __builtin_fma(double(r[i] & 0xFFFFu), wh_of(wh, r[i]), p);
    ent = open ? r[i] : ent;
  }
  if (!(xs < p)) {
#pragma unroll
    for (int i = 0; i < kRun; ++i)
      if ((r[i] & 0xFFFFu) != 0u && wh_of(wh, r[i]) > 0.0) ent = r[i];
  }
  return ent;
}

// The lane's index in the wave, computed where it is used: an opaque value
// keeps the compiler from hoisting the many lane-derived offsets and masks of
// the rounds out of the loops, where they would all stay live and spill.
__device__ __forceinline__ int lane_here() {
  int v;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(v));
  return v;
}

// Codes left in a token's topic slot by the small-group rounds: the draw
// fell in S' (the entry is found by a walk over the recorded run) or in Q'
// (a search of the word's Q' prefix).  Topics are below 2^15.
constexpr uint16_t kDrawS = 0xFFFF;
constexpr uint16_t kDrawQ = 0xFFFE;

// Topic of x in [0, Q') by the word's Q' prefix: the block by a binary
// search of qb (blocks of kGroup topics, +inf past the last), then a walk
// over the block's alpha * W^' terms (W^' is 0 from K up to the block end).  A rounding that leaves x at or past
// the end selects the last positive term.
__device__ __forceinline__ uint32_t q_draw(double xq, const WordState &w) {
  if (!(xq < w.qb[w.nb])) return (w.K1 == uint32_t(w.K - 1)) ? uint32_t(w.K - 2) : uint32_t(w.K - 1);
  int lo = 0;  // the largest block with qb[lo] <= xq (qb is +inf from nb + 1 up to 2 * qhalf)
  for (int step = w.qhalf; step > 0; step >>= 1) lo = w.qb[lo + step] <= xq ? lo + step : lo;
  const double xs = xq - w.qb[lo];
  if (w.qw) {
    // the walk below, by a binary search over the same partial sums (kept
    // per region): the last topic whose partial sum before it is <= xs
    const double *pw = w.qw + lo * kQwStride;
    if (!(xs < pw[kGroup])) return uint32_t(lo * kGroup + w.ql[lo]);
    int i = 0;
#pragma unroll
    for (int step = kGroup / 2; step > 0; step >>= 1) i = pw[i + step] <= xs ? i + step : i;
    return uint32_t(lo * kGroup + i);
  }
  const int k0 = lo * kGroup;
  double p = 0.0;
  int kk = k0, last = k0;
#pragma unroll
  for (int i = 0; i < kGroup; ++i) {
    const int k = k0 + i;
    const double t = w.alpha * w.wh[k];  // zeros past K (the row is padded to whole blocks)
    const bool open = p <= xs;
    p += t;
    kk = open ? k : kk;
    last = t > 0.0 ? k : last;
  }
  return uint32_t(xs < p ? kk : last);
}

// The drawn topic of a batch token, one lane per token: the topic itself,
// or the end of an S' or Q' draw recorded by the rounds.
__device__ __forceinline__ uint32_t finish_draw(int q, const BatchLds &bt, const WordState &w,
                                                const uint32_t *__restrict__ d_ent) {
  const uint32_t code = bt.top[q];
  if (code == kDrawS) {
    const uint32_t a = bt.off[q];
    uint32_t r[kRun];
    load_run<kRun>(d_ent + (a & ~uint32_t(kRun - 1)), 0, r);
    if (a & 1u) r[0] = uint32_t(w.K) << 16;  // the run starts with the row header
    return walk_run(r, w.wh, bt.u[q]) >> 16;
  }
  if (code == kDrawQ) return q_draw(bt.u[q], w);
  return code;
}

// One round of small-group draws: group g of the wave draws the token in
// list slot `slot` (if slot < n).  The row is read in chunks of G*kRun
// entries, lane l holding entries [l*kRun, l*kRun + kRun) of each chunk (the
// group's loads of a chunk share cache lines); NC is the largest chunk count
// in the round, and a group whose row has fewer chunks skips the rest.
// Sum: no draw; bt.u of the token gets the sum of its row's terms.
template <int G, int NC, bool Sum>
__device__ void draw_small(const BatchLds &bt, int slot, int n, const WordState &w,
                           const uint32_t *__restrict__ d_ent, int li, uint32_t &after_s) {
  constexpr uint32_t kSpan = uint32_t(G) * kRun;  // entries per chunk
  bool in_m = false;
  if (slot < n) {
    const int src = bt.list[slot];
    const uint32_t nc = (bt.nnz[src] + 1u + kSpan - 1) / kSpan;  // slots: header + entries
    const uint32_t off0 = bt.off[src];
    const uint32_t *run = d_ent + off0 + uint32_t(li) * kRun;
    const uint32_t pad = uint32_t(w.K) << 16;
    const double u = bt.u[src];
    // pass over the row: every chunk's loads are issued before the first is
    // used (one memory latency per row, not one per chunk); then per lane
    // and chunk the S' sum of kRun entries, and C1
    uint32_t r[NC][kRun];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      if (uint32_t(c) < nc) load_run<kRun>(run + c * kSpan, 0, r[c]);
    }
    if (li == 0) r[0][0] = pad;  // the row header
    double s[NC], T[NC];
    uint32_t c1 = 0xFFFFFFFFu;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      s[c] = 0.0;
      if (uint32_t(c) < nc) {
        if (!Sum) c1 = run_count_of<kRun>(r[c], w.K1, c1);
        s[c] = run_sum<kRun>(r[c], w.wh);
      }
    }
    // group totals, cumulative over the chunks (a missing chunk adds 0)
    double S = 0.0;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      S += gsum<G>(s[c]);
      T[c] = S;
    }
    if constexpr (Sum) {
      if (li == 0) bt.u[src] = S;
      return;
    }
    c1 = gmin_u32<G>(c1);
    // max-topic branch, Eq. 7: M = W^[v][K1] * (D[d][K1] + alpha)
    const double Mm = w.a1 * (double(c1 <= 0xFFFFu ? c1 : 0u) + w.alpha);
    const double x = u * ((Mm + S) + w.qp);
    in_m = x < Mm;
    if (!in_m) {
      if (x < Mm + S) {
        // S': the chunk (the first whose cumulative total passes x; it has a
        // positive total), the lane, then the entry
        int cs = 0;
        double base = Mm, sc = s[0];
#pragma unroll
        for (int c = 1; c < NC; ++c) {
          if (uint32_t(c) < nc && x >= Mm + T[c - 1]) {
            cs = c;
            base = Mm + T[c - 1];
            sc = s[c];
          }
        }
        const double incl = gscan<G>(sc, li);
        const int sel = pick_lane<G>(sc, incl, base, x, li);
        if (li == sel) {
          // the selected lane's run and x inside it, for the walk after the rounds
          bt.off[src] = (off0 + uint32_t(cs) * kSpan + uint32_t(li) * kRun) | (cs == 0 && li == 0 ? 1u : 0u);
          bt.u[src] = fmax(x - (base + (incl - sc)), 0.0);
          bt.top[src] = kDrawS;
        }
      } else if (li == 0) {
        // Q': x past M + S', searched after the rounds
        bt.u[src] = x - (Mm + S);
        bt.top[src] = kDrawQ;
      }
    }
    if (in_m && li == 0) bt.top[src] = uint16_t(w.K1);
  }
  // outside the divergent part, so the count stays wave-uniform
  if (!Sum) after_s += uint32_t(__popcll(__ballot(in_m && li == 0)));
}

// Row-length buckets of a batch (slots, header included): upper bounds.
// Buckets 0-3 are rows padded to 32-slot multiples, 4-5 to 64, 6-7 to 128.
__device__ constexpr uint32_t kBucketEnd[8] = {32, 64, 96, 128, 192, 256, 384, 512};

// The small-group rounds over list places [from, to) (rows in ascending
// bucket order), G lanes per token and 64/G tokens a round.  A round reads
// as many chunks of G*kRun slots as its last (longest) row needs.
template <int G, int MaxNC, bool Sum>
__device__ void draw_rounds(int from, int to, const int (&ends)[8], const BatchLds &bt, const WordState &w,
                            const uint32_t *__restrict__ d_ent, uint32_t &after_s) {
  constexpr uint32_t kSpan = uint32_t(G) * kRun;
  for (int base = from; base < to; base += kWave / G) {
    const int ln = lane_here(), g = ln / G, li = ln % G;
    const int last = min(base + kWave / G, to) - 1;
    uint32_t upper = kBucketEnd[7];
#pragma unroll
    for (int k = 6; k >= 0; --k) upper = last < ends[k] ? kBucketEnd[k] : upper;
    const uint32_t nc = (upper + kSpan - 1) / kSpan;
    const int slot = base + g;
    if (nc <= 1) {
      draw_small<G, 1, Sum>(bt, slot, to, w, d_ent, li, after_s);
    } else if (nc == 2) {
      draw_small<G, 2, Sum>(bt, slot, to, w, d_ent, li, after_s);
    } else if (nc == 3) {
      draw_small<G, 3, Sum>(bt, slot, to, w, d_ent, li, after_s);
    } else if (MaxNC <= 4 || nc == 4) {
      draw_small<G, 4, Sum>(bt, slot, to, w, d_ent, li, after_s);
    } else {
      if constexpr (MaxNC > 4) {
        if (nc <= 6) draw_small<G, 6, Sum>(bt, slot, to, w, d_ent, li, after_s);
        else draw_small<G, MaxNC, Sum>(bt, slot, to, w, d_ent, li, after_s);
      }
    }
  }
}

// The small-group draws of one batch.  The lanes left to draw are listed in
// ascending bucket order; rows of up to 128 slots are drawn by groups of 4
// lanes (16 a round), up to 256 by 8 lanes, up to 512 by 16 lanes.  When the
// 4-lane rounds would end with a partial round of at most 8 rows, all of
// 97-128 slots (two whole 64-slot chunks), those rows join the 8-lane
// rounds instead: they fill free places there, or make a round that reads
// half as many entries per lane as the partial 4-lane round would.
// Wide (sums only: the LLPT kernel's 1,024-thread workgroups, whose waves have
// registers to spare): rows of up to 512 slots by 8 lanes as well, 8 tokens a
// round, so that a round's per-token work (sums, scans) serves twice the
// tokens.
template <bool Wide, bool Sum>
__device__ void draw_batch_small(bool und, uint32_t nnz, const BatchLds &bt, const WordState &w,
                                 const uint32_t *__restrict__ d_ent, int lane, uint32_t &after_s) {
  static_assert(Sum || !Wide, "no workgroup of 1,024 threads draws in fp64");
  int n = 0, ends[8];
  const uint32_t slots = nnz + 1u;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const uint32_t lo = k ? kBucketEnd[k - 1] : 0u;
    const unsigned long long m = __ballot(und && slots > lo && slots <= kBucketEnd[k]);
    if ((m >> lane) & 1ull)
      bt.list[n + int(__builtin_amdgcn_mbcnt_hi(uint32_t(m >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(m), 0u)))] =
          uint8_t(lane);
    n += __popcll(m);
    ends[k] = n;
  }
  const int left = ends[3] % 16;
  const int a = left > 0 && left <= 8 && ends[3] - ends[2] >= left ? ends[3] - left : ends[3];
  draw_rounds<4, 4, Sum>(0, a, ends, bt, w, d_ent, after_s);
  if (Wide) {
    draw_rounds<8, 8, Sum>(a, ends[7], ends, bt, w, d_ent, after_s);
  } else {
    draw_rounds<8, 4, Sum>(a, ends[5], ends, bt, w, d_ent, after_s);
    draw_rounds<16, 4, Sum>(ends[5], ends[7], ends, bt, w, d_ent, after_s);
  }
}

// The draws of the lanes with `und` set: lane ln holds the token staged in
// slot ln of the batch (row offset off, row length nnz); lanes before `first`
// belong to another word.  Returns the drawn topic per lane (und lanes only);
// *nnz_read gets the D-row entries this lane's draw reads.
// Long rows: runs of tokens of one document (same row offset), whose later
// tokens draw from the sums of the run's first one.  Rows of up to 128 slots
// (header and entries): 4 lanes per token; up to 256: 8 lanes; up to 512: 16
// lanes; longer rows: 16 lanes, one chunk of kChunk slots at a time; then the
// S' walks and Q' searches, one lane per token.
// Sum: no draws; bt.u of every such lane gets the sum of its row's terms
// D[d][k] * W^[v][k] instead (w.wh with all of W^[v]).
template <bool Wide = false, bool Sum = false>
__device__ __forceinline__ uint32_t draw_tokens(bool und, uint32_t off, uint32_t nnz, int first, int ln,
                                                const BatchLds &bt, const WordState &w,
                                                const uint32_t *__restrict__ d_ent, uint32_t &after_s,
                                                uint32_t *nnz_read) {
  const unsigned long long lmask = __ballot(und && nnz + 1u > 512u);
  unsigned long long starts = 0ull;
  bool fol = false;
  if (lmask) {
    const uint32_t prev_off = uint32_t(__shfl(int(off), ln - 1));
    starts = __ballot(ln == first || off != prev_off);
    const unsigned long long below = ln ? ~0ull >> (64 - ln) : 0ull;
    const int rs = 63 - __clzll((long long)(starts & (below | (1ull << ln))));  // this lane's run start
    fol = ((lmask >> ln) & 1ull) && (lmask & below & (~0ull << rs)) != 0ull;
  }
  *nnz_read = und ? (fol ? min(nnz, uint32_t(kChunk)) : nnz) : 0u;  // a follower reads one chunk of its row
  draw_batch_small<Wide, Sum>(und, nnz, bt, w, d_ent, ln, after_s);
  if (lmask) draw_long<Sum>(lmask, __ballot(fol), starts, bt, w, d_ent, ln / kGroup, ln % kGroup, after_s);
  if (Sum) return 0u;
  return und ? finish_draw(ln, bt, w, d_ent) : 0u;
}

// One wave's statistics (lane 0 stores them); first: the workgroup's first
// wave, which also stores the regions' counts.
__device__ __forceinline__ void store_stats(const DevState &d, uint32_t slot, bool first, uint32_t sampled,
                                            uint32_t after_s, unsigned long long nnz, uint32_t regions,
                                            uint32_t dense_regions, unsigned long long row_bytes) {
  unsigned long long *st = d.wave_stats + slot;
  st[size_t(WV_SAMPLED) * kWaveSlots] = sampled;
  st[size_t(WV_AFTER_S) * kWaveSlots] = after_s;
  st[size_t(WV_NNZ) * kWaveSlots] = nnz;
  st[size_t(WV_REGIONS) * kWaveSlots] = first ? regions : 0u;
  st[size_t(WV_DENSE_REGIONS) * kWaveSlots] = first ? dense_regions : 0u;
  st[size_t(WV_ROW_BYTES) * kWaveSlots] = first ? row_bytes : 0ull;
}

// The sampler with the W^' row in fp64 (K below kF32Topics): workgroups of four
// waves that share a word's row in LDS, every wave on its own batches.  It
// takes the units (sampler_units) of the regions before p.light_begin; the
// light regions are k_sampler_light's.
__global__ __launch_bounds__(kBlock, 7) void k_sampler(DevState d, Params p, uint32_t t,
                                                       unsigned long long *__restrict__ stats) {
  extern __shared__ double lds[];
  constexpr int NB = kBlock;
  const int K = p.K;
  const int nb = (K + kGroup - 1) / kGroup;
  const int nbp = q_blocks_padded(nb);
  const bool by_doc = doc_marks(d, p, t);  // which bitmap carries this iteration's skip decisions
  // dynamic LDS only (sampler_lds_bytes)
  double *wh = lds;                  // [wh_entries(K)]: W^' of the region's word, zeros past K
  double *qb = lds + wh_entries(K);  // [nbp + 1]: qb[b] = sum of alpha*W^' over topics < b*kGroup; +inf past nb
  double *s_u = qb + nbp + 1;        // [NB]: the batch slices of the waves
  uint32_t *s_off = reinterpret_cast<uint32_t *>(s_u + NB);  // [NB]
  uint32_t *s_nnz = s_off + NB;                              // [NB]
  uint32_t *s_hand = s_nnz + NB;                             // [NB / kGroup * kMaxRun]
  uint32_t *s_reg = s_hand + NB / kGroup * kMaxRun;          // [4]: the region (word, begin, end) and a valid flag
  uint16_t *s_top = reinterpret_cast<uint16_t *>(s_reg + 4); // [NB]
  uint8_t *s_list = reinterpret_cast<uint8_t *>(s_top + NB); // [NB]
  // with p.q_table: [nb * kQwStride] partial sums of the Q' blocks, then [nb] last-positive offsets
  // (the 21 * NB + 16 bytes after s_u keep them 8-byte aligned)
  static_assert((21 * NB + 16) % 8 == 0, "the Q' partial sums must be 8-byte aligned");
  double *s_qw = p.q_table ? reinterpret_cast<double *>(s_list + NB) : nullptr;
  uint8_t *s_ql = p.q_table ? reinterpret_cast<uint8_t *>(s_qw + nb * kQwStride) : nullptr;

  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  if (blockIdx.x == 0 && tid == 0) stats[ST_MARKS] = by_doc ? 2ull : 1ull;
  const BatchLds bt{s_off + wave * kWave, s_nnz + wave * kWave, s_u + wave * kWave, s_top + wave * kWave,
                    s_hand + wave * (kWave / kGroup) * kMaxRun, s_list + wave * kWave};
  const int qhalf = nbp / 2;
  for (int q = nb + 1 + tid; q < nbp; q += NB) qb[q] = __builtin_inf();
  for (int k = K + 1 + tid; k < wh_entries(K); k += NB) wh[k] = 0.0;
  // region, word and count variables are uniform over the block (scalar registers)
  uint32_t cur = 0xFFFFFFFFu, K1 = 0;
  double a1 = 0.0, qp = 0.0;
  // the sparse word whose row wh holds (null if a dense row or none): the
  // next sparse word only restores that word's topics and K1 to beta/den[k]
  const uint32_t *held = nullptr;
  uint32_t held_nnz = 0, held_k1 = 0;
  // (tokens of a corpus, and so these counts, fit 32 bits)
  uint32_t n_sampled = 0, n_after_s = 0, n_reg = 0, n_dreg = 0;
  unsigned long long nnz_sum = 0, row_bytes = 0;

  for (;;) {
    if (tid == 0) {
      const int64_t r = int64_t(atomicAdd(&d.counters[CNT_SAMPLER], 1u));
      s_reg[3] = r < p.n_units ? 1u : 0u;
      if (s_reg[3]) {
        s_reg[0] = d.unit[3 * size_t(r)];
        s_reg[1] = d.unit[3 * size_t(r) + 1];
        s_reg[2] = d.unit[3 * size_t(r) + 2];
      }
    }
    __syncthreads();
    if (!s_reg[3]) break;
    const uint32_t vc = __builtin_amdgcn_readfirstlane(s_reg[0]), v = vc & ~kUnitContinues;
    const uint32_t b = __builtin_amdgcn_readfirstlane(s_reg[1]);
    const uint32_t e = __builtin_amdgcn_readfirstlane(s_reg[2]);
    if (vc == v) {  // the first unit of its region
      n_reg++;
      if (int32_t(v) < p.n_dense) n_dreg++;
    }
    if (b == d.word_off[v])
      row_bytes += int32_t(v) < p.n_dense ? 4ull * uint64_t(K) : 4ull * d.ws_nnz[int(v) - p.n_dense];
    if (v != cur) {
      cur = v;
      const WordRec rec = d.wrec[v];
      K1 = rec.k1;
      a1 = rec.a1;
      qp = rec.qp;
      if (int32_t(v) < p.n_dense) {
        const int32_t *wrow = d.w_dense + size_t(v) * size_t(K);
        for (int k = tid; k < K; k += NB) wh[k] = what(uint32_t(wrow[k]), p.beta, d.den[k]);
        held = nullptr;
      } else {
        const int s = int(v) - p.n_dense;
        const uint32_t *ents = d.ws_ent + d.ws_cap[s];
        const uint32_t nnz = d.ws_nnz[s];
        if (held) {
          for (uint32_t q = tid; q < held_nnz; q += NB) {
            const uint32_t k = held[q] >> 16;
            wh[k] = d.bden[k];
          }
          if (tid == 0 && held_k1 < uint32_t(K)) wh[held_k1] = d.bden[held_k1];  // K1 = K in two-branch mode
        } else {
          for (int k = tid; k < K; k += NB) wh[k] = d.bden[k];
        }
        __syncthreads();
        for (uint32_t q = tid; q < nnz; q += NB) {
          const uint32_t ent = ents[q];
          wh[ent >> 16] = what(ent & 0xFFFFu, p.beta, d.den[ent >> 16]);
        }
        held = ents;
        held_nnz = nnz;
        held_k1 = K1;
      }
      __syncthreads();
      // the max topic is its own branch: W^' has a 0 there (Eq. 5)
      if (tid == 0) {
        wh[K1] = 0.0;
        wh[K] = 0.0;  // topic of the padding entries of D rows
      }
      __syncthreads();
      // the Q' prefix over blocks of kGroup topics: thread i sums blocks i,
      // i + NB, ..., then per round a scan per wave (DPP) leaves the block's
      // prefix inside its wave in qb and the wave's total in s_u; after the
      // barrier each block adds the totals before its wave, in round and wave
      // order.  Without the partial-sum table a block is summed from topic
      // i % 16 on, wrapping, so that the 16 lanes of a row read 16 different
      // LDS bank pairs (wh past K holds zeros).
      double *s_tot = s_u;  // [rounds * waves <= NB]; s_u is next written by the token batches
      uint32_t rot;         // i % 16, opaque to the compiler: otherwise it keeps the 16 rotated addresses live
      asm volatile("v_mov_b32 %0, %1" : "=v"(rot) : "v"(uint32_t(lane & (kGroup - 1))));
      for (int r = 0; r * NB < nb; ++r) {
        const int blk = r * NB + tid;
        double s = 0.0;
        if (blk < nb) {
          if (s_qw) {
            // every topic of the block (zeros past K), as q_draw's walk adds them
            double *pw = s_qw + blk * kQwStride;
            int last = 0;
            for (int i = 0; i < kGroup; ++i) {
              pw[i] = s;
              const double t = p.alpha * wh[blk * kGroup + i];
              s += t;
              last = t > 0.0 ? i : last;
            }
            pw[kGroup] = s;
            s_ql[blk] = uint8_t(last);
          } else {
            const double *wb = wh + blk * kGroup;
#pragma unroll
            for (uint32_t i = 0; i < uint32_t(kGroup); ++i) s += p.alpha * wb[(i + rot) & uint32_t(kGroup - 1)];
          }
        }
        const double incl = wave_incl_scan(s);
        if (blk < nb) qb[blk + 1] = incl;
        if (lane == kWave - 1) s_tot[r * (NB / kWave) + wave] = incl;
      }
      __syncthreads();
      {
        double acc = 0.0;
        for (int r = 0; r * NB < nb; ++r) {
          double own = 0.0;
          for (int w = 0; w < NB / kWave; ++w) {
            if (w == wave) own = acc;
            acc += s_tot[r * (NB / kWave) + w];
          }
          const int blk = r * NB + tid;
          if (blk < nb) qb[blk + 1] = own + qb[blk + 1];
        }
        if (tid == 0) qb[0] = 0.0;
      }
      __syncthreads();
    }

    const WordState w{wh, qb, nb, K, qhalf, K1, a1, qp, p.alpha, s_qw, s_ql};
    // tokens per batch: 64, or fewer when the region has too few tokens to
    // give every wave a whole batch, so that a small region's batches (each
    // a chain of dependent loads and rounds) run side by side on several
    // waves instead of one after another on one
    const uint32_t bsz = min(uint32_t(kWave), max(16u, ((e - b + uint32_t(NB / kWave) - 1u) / uint32_t(NB / kWave) + 15u) & ~15u));
    for (uint32_t base = b + uint32_t(wave) * bsz; base < e; base += uint32_t(NB / kWave) * bsz) {
      const int ln = lane_here();  // the lane, recomputed per batch
      const uint32_t j = base + uint32_t(ln);
      const uint32_t be = min(e, base + bsz);  // the batch's end
      // the slot, key and row offset are loaded together (one latency); the
      // row header only for the tokens left to draw
      uint32_t sk = 0, key = 0, off = 0;
      if (j < be) {
        const uint2 kr = d.wt_kr[j];
        key = kr.x;
        off = kr.y;  // the row's first slot (its header)
        // the skip bit at the word-order slot, or at the key (the token's
        // document position) in the document-ordered bitmap
        sk = by_doc ? d.skip_doc[key >> 5] >> (key & 31u) : d.skip_bits[j >> 5] >> (j & 31u);
      }
      const bool und = j < be && !(sk & 1u);
      uint32_t nnz = 0;
      if (und) {
        nnz = d.d_ent[off] & 0xFFFFu;
        bt.off[ln] = off;
        bt.nnz[ln] = nnz;
        bt.u[ln] = uniform_draw(p.seed, t, key);
      }
      n_sampled += uint32_t(__popcll(__ballot(und)));
      uint32_t nnz_read;
      const uint32_t drawn = draw_tokens(und, off, nnz, 0, ln, bt, w, d.d_ent, n_after_s, &nnz_read);
      nnz_sum += wave_sum_u32(nnz_read);
      // the batch's topics (K1 for the tokens the step-3 test decided) leave in one coalesced store
      const uint32_t topic = und ? drawn : K1;
      if (j < be) d.z_w[j] = uint16_t(topic);
    }
    __syncthreads();
  }
  if (lane == 0)
    store_stats(d, blockIdx.x * uint32_t(NB / kWave) + uint32_t(wave), wave == 0, n_sampled, n_after_s, nnz_sum, n_reg,
                n_dreg, row_bytes);
}

// W^ of a dense row into a wave's LDS row, kLightAhead topics per lane loaded
// together (one after another each topic waited for memory: out of core, where
// every light word is a dense row, 1.20 ms a chunk of 123,000 words).
constexpr int kLightAhead = 8;
__device__ __forceinline__ void fill_dense_wave(const int32_t *__restrict__ wrow, const double *__restrict__ den,
                                                double beta, int K, int lane, double *__restrict__ wh) {
  for (int k0 = lane; k0 < K; k0 += kLightAhead * kWave) {
    uint32_t c[kLightAhead];
    double dn[kLightAhead];
#pragma unroll
    for (int u = 0; u < kLightAhead; ++u) {
      const int k = min(k0 + u * kWave, K - 1);
      c[u] = uint32_t(wrow[k]);
      dn[u] = den[k];
    }
#pragma unroll
    for (int u = 0; u < kLightAhead; ++u)
      if (k0 + u * kWave < K) wh[k0 + u * kWave] = what(c[u], beta, dn[u]);
  }
}

// The light regions (Sec. 5.1: light units to wavefronts): words of at most
// kLightTokens tokens, the suffix [p.light_begin, n_regions) of the region
// table.  A wave takes batches of consecutive light words (d.light_batch: at
// most 64 tokens together), dealt round-robin over the grid.  The tokens of
// all the batch's words are staged at once, one per lane (records, row header
// and uniform), then the words are drawn in turn: the W^' row in the wave's
// LDS with only the previous word's topics restored, the Q' prefix, the
// rounds over the word's lanes.  The next word's row entries are loaded while
// a word is drawn.
//
// What bounds it is the chain of memory latencies per word, so the wave holds
// as little LDS as it can (no table of the Q' blocks' partial sums: 16 waves
// per CU at K = 1,000 instead of 8) and no word waits for a counter: a
// counter on one address takes about 85 million atomics a second, 7.3 ms for
// 623,000 light words.
__global__ __launch_bounds__(64, 4) void k_sampler_light(DevState d, Params p, uint32_t t,
                                                         unsigned long long *__restrict__ stats) {
  extern __shared__ double lds[];
  const int K = p.K;
  const int nb = (K + kGroup - 1) / kGroup;
  const int nbp = q_blocks_padded(nb);
  const bool by_doc = doc_marks(d, p, t);
  double *wh = lds;                  // [wh_entries(K)]
  double *qb = lds + wh_entries(K);  // [nbp + 1]
  double *s_u = qb + nbp + 1;        // [64]
  uint32_t *s_off = reinterpret_cast<uint32_t *>(s_u + kWave);
  uint32_t *s_nnz = s_off + kWave;
  uint32_t *s_hand = s_nnz + kWave;  // [kWave / kGroup * kMaxRun]
  uint16_t *s_top = reinterpret_cast<uint16_t *>(s_hand + kWave / kGroup * kMaxRun);
  uint8_t *s_list = reinterpret_cast<uint8_t *>(s_top + kWave);
  const BatchLds bt{s_off, s_nnz, s_u, s_top, s_hand, s_list};
  const int lane = threadIdx.x;
  if (blockIdx.x == 0 && lane == 0) stats[ST_MARKS] = by_doc ? 2ull : 1ull;
  for (int q = nb + 1 + lane; q < nbp; q += kWave) qb[q] = __builtin_inf();
  if (lane == 0) qb[0] = 0.0;
  for (int k = K + lane; k < wh_entries(K); k += kWave) wh[k] = 0.0;
  // the sparse word whose row wh holds: its entries (held < 0: a dense row or
  // none, so that all of wh is rewritten), lane q the topic of entry q and its
  // beta/den, and K1 with what wh had there
  int held = -1;
  uint32_t held_k = 0, held_k1 = 0;
  double held_b = 0.0, held_w1 = 0.0;
  uint32_t n_sampled = 0, n_after_s = 0, n_reg = 0, n_dreg = 0;
  unsigned long long nnz_sum = 0, row_bytes = 0;
  // a wave's LDS accesses run in order; the fence keeps the compiler's order
  auto order = [&]() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); };

  for (uint32_t bi = blockIdx.x; bi < uint32_t(p.n_light_batches); bi += gridDim.x) {
    const uint32_t r0 = __builtin_amdgcn_readfirstlane(d.light_batch[bi]);
    const int nw = int(__builtin_amdgcn_readfirstlane(d.light_batch[bi + 1]) - r0);  // 1..64
    // lane i: word i of the batch
    const size_t rr = 3 * (size_t(p.light_begin) + r0 + uint32_t(min(lane, nw - 1)));
    const uint32_t v_l = d.region[rr], b_l = d.region[rr + 1], e_l = d.region[rr + 2];
    const uint32_t b0 = __builtin_amdgcn_readlane(b_l, 0), e0 = __builtin_amdgcn_readlane(e_l, nw - 1);
    // lane ln: token ln of the batch
    const int ln = lane_here();
    const uint32_t j = b0 + uint32_t(ln);
    uint32_t sk = 0, key = 0, off = 0;
    if (j < e0) {
      const uint2 kr = d.wt_kr[j];
      key = kr.x;
      off = kr.y;
      sk = by_doc ? d.skip_doc[key >> 5] >> (key & 31u) : d.skip_bits[j >> 5] >> (j & 31u);
    }
    const bool und = j < e0 && !(sk & 1u);
    const bool dense_l = int32_t(v_l) < p.n_dense;
    const int s_l = dense_l ? 0 : int(v_l) - p.n_dense;
    const uint32_t nnz_l = dense_l ? 0u : d.ws_nnz[s_l];
    const uint32_t cap_l = dense_l ? 0u : d.ws_cap[s_l];
    const uint32_t k1_l = d.wrec[v_l].k1;
    const double a1_l = d.wrec[v_l].a1, qp_l = d.wrec[v_l].qp;
    uint32_t nnz = 0;
    if (und) {
      nnz = d.d_ent[off] & 0xFFFFu;
      bt.off[ln] = off;
      bt.nnz[ln] = nnz;
      bt.u[ln] = uniform_draw(p.seed, t, key);
    }
    n_sampled += uint32_t(__popcll(__ballot(und)));
    n_reg += uint32_t(nw);
    n_dreg += uint32_t(__popcll(__ballot(lane < nw && dense_l)));
    if (lane < nw && b_l == d.word_off[v_l]) row_bytes += dense_l ? 4ull * uint64_t(K) : 4ull * nnz_l;
    // word i's row entry (one per lane: a sparse word of at most 64 tokens)
    auto entry_of = [&](int i) {
      const uint32_t n = __builtin_amdgcn_readlane(nnz_l, i), c = __builtin_amdgcn_readlane(cap_l, i);
      return uint32_t(lane) < n ? d.ws_ent[c + uint32_t(lane)] : 0u;
    };
    // loaded ahead of their use, so that no word waits for them: the entries
    // two words ahead, den and beta/den of their topics one word ahead
    uint32_t ent_1 = entry_of(0), ent_2 = entry_of(min(1, nw - 1));
    double den_1 = d.den[ent_1 >> 16], bden_1 = d.bden[ent_1 >> 16];
    uint32_t topic = 0;
    for (int i = 0; i < nw; ++i) {
      const uint32_t v = __builtin_amdgcn_readlane(v_l, i);
      const uint32_t ent = ent_1;
      const double den_e = den_1, bden_e = bden_1;
      ent_1 = ent_2;
      den_1 = d.den[ent_1 >> 16];
      bden_1 = d.bden[ent_1 >> 16];
      ent_2 = entry_of(min(i + 2, nw - 1));
      const int f = int(__builtin_amdgcn_readlane(b_l, i) - b0), l = int(__builtin_amdgcn_readlane(e_l, i) - b0);
      const uint32_t K1 = __builtin_amdgcn_readlane(k1_l, i);
      const bool mine = ln >= f && ln < l;
      if (__ballot(mine && und) == 0ull) {  // decided by step 3
        if (mine) topic = K1;
        continue;
      }
      const double a1 = readlane_f64(a1_l, i), qp = readlane_f64(qp_l, i);
      if (int32_t(v) < p.n_dense) {
        const int32_t *wrow = d.w_dense + size_t(v) * size_t(K);
        fill_dense_wave(wrow, d.den, p.beta, K, lane, wh);
        held = -1;
      } else {
        const uint32_t n = __builtin_amdgcn_readlane(nnz_l, i);
        const uint32_t ek = ent >> 16;
        const double we = uint32_t(lane) < n ? what(ent & 0xFFFFu, p.beta, den_e) : 0.0;
        if (held >= 0) {
          if (lane == 0) wh[held_k1] = held_w1;  // before the row: K1 may be in it
          order();
          if (lane < held) wh[held_k] = held_b;
        } else {
          for (int k = lane; k < K; k += kWave) wh[k] = d.bden[k];
        }
        order();
        if (uint32_t(lane) < n) wh[ek] = we;
        held = int(n);
        held_k = ek;
        held_b = bden_e;
        held_k1 = K1;
      }
      order();
      if (lane == 0) {
        held_w1 = wh[K1];
        wh[K1] = 0.0;  // the max topic is its own branch (Eq. 5)
        wh[K] = 0.0;   // topic of the padding entries of D rows
      }
      order();
      // the Q' prefix over blocks of kGroup topics, one block per lane and
      // round, summed from topic lane % 16 on, wrapping, so that the 16 lanes
      // of a row read 16 different LDS bank pairs
      uint32_t rot;
      asm volatile("v_mov_b32 %0, %1" : "=v"(rot) : "v"(uint32_t(ln & (kGroup - 1))));
      double acc = 0.0;
      for (int q0 = 0; q0 < nb; q0 += kWave) {
        const int blk = q0 + ln;
        double s = 0.0;
        if (blk < nb) {
          const double *wb = wh + blk * kGroup;
#pragma unroll
          for (uint32_t q = 0; q < uint32_t(kGroup); ++q) s += p.alpha * wb[(q + rot) & uint32_t(kGroup - 1)];
        }
        const double incl = acc + wave_incl_scan(s);
        if (blk < nb) qb[blk + 1] = incl;
        acc = __shfl(incl, kWave - 1);
      }
      order();
      const WordState w{wh, qb, nb, K, nbp / 2, K1, a1, qp, p.alpha, nullptr, nullptr};
      uint32_t nnz_read;
      const uint32_t drawn = draw_tokens(mine && und, off, nnz, f, ln, bt, w, d.d_ent, n_after_s, &nnz_read);
      nnz_sum += wave_sum_u32(nnz_read);
      if (mine) topic = und ? drawn : K1;
      order();  // wh and qb are rewritten for the next word
    }
    if (j < e0) d.z_w[j] = uint16_t(topic);
  }
  row_bytes = group_sum_u64<kWave>(row_bytes);
  if (lane == 0)
    store_stats(d, uint32_t(stat_slots(p, t).light0) + blockIdx.x, true, n_sampled, n_after_s, nnz_sum, n_reg, n_dreg,
                row_bytes);
}

// ---------------------------------------------------------- large K ----
// When the fp64 W^ row does not fit in LDS (K above about 17,000 topics, up to
// 32,768), the LLPT kernel (k_loglik_tiled) splits the topics in two tiles,
// [0, KT) and [KT, K] (topic K is the padding of D rows), and walks a region
// twice.  Entries of the other tile read a zero.
struct TileState {
  const double *wt;  // the tile: W^' of topics [base, base + KT), zeros past the tile's end
  uint32_t base, kt;
  uint32_t rel;      // -base * 8 (mod 2^32)
};

// W^' of a packed D entry's topic if it lies in the tile, else 0 (wt[kt] is
// 0).  The tile starts at LDS address 0 (the kernel's LDS is all dynamic,
// which launch_loglik checks), so the address (topic - base) * 8 is one
// v_mad_u32_u16 on the entry's high half; topics below the tile wrap to
// addresses near 2^32, and one unsigned min sends every topic outside the
// tile to wt[kt].
__device__ __forceinline__ double wt_of(const TileState &ts, uint32_t e) {
  uint32_t a;
  asm("v_mad_u32_u16 %0, %1, 8, %2 op_sel:[1,0,0,0]" : "=v"(a) : "v"(e), "s"(ts.rel));
  return *(lds_f64 *)(size_t)min(a, ts.kt * 8u);
}

// This lane's run of chunk ch of a row of `slots` padded slots; runs past
// the row read the padding entry, and the header (slot 0) is padding too.
__device__ __forceinline__ void load_run_masked(const uint32_t *__restrict__ row, uint32_t ch, uint32_t slots, int li,
                                                uint32_t pad, uint32_t (&r)[kMaxRun]) {
  const uint32_t q0 = ch * kChunk + uint32_t(li) * kMaxRun;
  if (q0 < slots) {
#pragma unroll
    for (int i = 0; i < kMaxRun; ++i) r[i] = row[q0 + i];
  } else {
#pragma unroll
    for (int i = 0; i < kMaxRun; ++i) r[i] = pad;
  }
  if (q0 == 0u) r[0] = pad;
}

__device__ __forceinline__ double run_sum_tile(const uint32_t (&r)[kMaxRun], const TileState &ts) {
  double s = 0.0;
#pragma unroll
  for (int i = 0; i < kMaxRun; ++i) s = __builtin_fma(double(r[i] & 0xFFFFu), wt_of(ts, r[i]), s);
  return s;
}

// Fills the tile [base, base + len) of the region's word (zeros elsewhere,
// at K1 and at the padding topic K).  Each thread issues the loads of
// kFillBatch topics (or row entries) before it uses the first, so that a
// fill waits on a few memory latencies rather than one per topic.
constexpr int kFillBatch = 8;
__device__ void fill_tile(const DevState &d, const Params &p, uint32_t v, uint32_t K1, uint32_t base, uint32_t len,
                          uint32_t kt, double *__restrict__ wt, int tid, int nthreads) {
  const uint32_t K = uint32_t(p.K), n = kt + uint32_t(kGroup), nt = uint32_t(nthreads);
  // loads at clamped (always valid) topics; the topics outside the tile get 0
  if (int32_t(v) < p.n_dense) {
    const int32_t *wrow = d.w_dense + size_t(v) * size_t(K);
    uint32_t q0 = uint32_t(tid);
    for (; q0 + (kFillBatch - 1) * nt < n; q0 += kFillBatch * nt) {
      uint32_t cnt[kFillBatch];
      double dn[kFillBatch];
#pragma unroll
      for (int u = 0; u < kFillBatch; ++u) {
        const uint32_t k = min(base + q0 + uint32_t(u) * nt, K - 1u);
        cnt[u] = uint32_t(wrow[k]);
        dn[u] = d.den[k];
      }
#pragma unroll
      for (int u = 0; u < kFillBatch; ++u) {
        const uint32_t q = q0 + uint32_t(u) * nt, k = base + q;
        wt[q] = q < len && k < K && k != K1 ? what(cnt[u], p.beta, dn[u]) : 0.0;
      }
    }
    for (; q0 < n; q0 += nt) {
      const uint32_t k = base + q0;
      wt[q0] = q0 < len && k < K && k != K1 ? what(uint32_t(wrow[k]), p.beta, d.den[k]) : 0.0;
    }
  } else {
    const int s = int(v) - p.n_dense;
    const uint32_t *ents = d.ws_ent + d.ws_cap[s];
    const uint32_t nnz = d.ws_nnz[s];
    uint32_t q0 = uint32_t(tid);
    for (; q0 + (kFillBatch - 1) * nt < n; q0 += kFillBatch * nt) {
      double bd[kFillBatch];
#pragma unroll
      for (int u = 0; u < kFillBatch; ++u) bd[u] = d.bden[min(base + q0 + uint32_t(u) * nt, K - 1u)];
#pragma unroll
      for (int u = 0; u < kFillBatch; ++u) {
        const uint32_t q = q0 + uint32_t(u) * nt, k = base + q;
        wt[q] = q < len && k < K && k != K1 ? bd[u] : 0.0;
      }
    }
    for (; q0 < n; q0 += nt) {
      const uint32_t k = base + q0;
      wt[q0] = q0 < len && k < K && k != K1 ? d.bden[k] : 0.0;
    }
    __syncthreads();
    for (uint32_t q0 = uint32_t(tid); q0 < nnz; q0 += kFillBatch * nt) {
      uint32_t ent[kFillBatch];
#pragma unroll
      for (int u = 0; u < kFillBatch; ++u) ent[u] = ents[min(q0 + uint32_t(u) * nt, nnz - 1u)];
      double dn[kFillBatch];
#pragma unroll
      for (int u = 0; u < kFillBatch; ++u) dn[u] = d.den[min(ent[u] >> 16, K - 1u)];
#pragma unroll
      for (int u = 0; u < kFillBatch; ++u) {
        const uint32_t k = ent[u] >> 16;
        if (q0 + uint32_t(u) * nt < nnz && k >= base && k < base + len && k < K && k != K1)
          wt[k - base] = what(ent[u] & 0xFFFFu, p.beta, dn[u]);
      }
    }
  }
  __syncthreads();
}

constexpr int kTiledBlock = 1024;           // threads per workgroup of k_loglik_tiled (16 waves)
constexpr int kTiledAhead = 2;              // chunks whose loads a group issues together

// ------------------------------------------------- certified draws ----
// The sampler with the W^' row in single precision.  The row is what limits
// the residency at large K (80 KB of fp64 at K = 10,000; 256 KB at 32,768,
// more than a CU has) and its gathers are the sampler's LDS traffic.  Half the
// size, it fits one workgroup at every K up to 32,768, and three workgroups
// of 512 threads at K = 10,000.
//
// No draw depends on the single precision.  S' and its prefixes are sums of
// nonnegative terms D[d][k] * W^[v][k]; a lane adds its run of 8 terms in
// fp32 (W^ rounded once, each fused multiply-add once) and everything else is
// fp64, so every prefix of S' is off by at most kEps of itself, kEps being a
// little over 9 * 2^-24.  With x = u*Z the draw is decided only when x is
// further than the bound on its own error and the edge's from both edges of
// the chosen segment; otherwise (2.4e-3 of the tokens at K = 10,000 and 5.7e-3
// at 32,768 in a fit's first iterations, 1.7e-3 and 3.6e-3 after 50, counted in
// a copy) a wave redoes the token with all of its arithmetic in fp64
// (exact_draw).  Either way the topic is the one the fp64 evaluation gives.
//   x against M and inside S': x - (M + prefix) is off by at most
//                              2 * e, e = kEps * S'
//   x inside Q':               x - (M + S') by at most (1 - u) * e, where
//                              1 - u < Q' / Z <= Q' / (S' + Q')
// tau = 2^-40 Z + 2^-90 on top covers the fp64 roundings (some 2^-50 of Z)
// and fp32 underflow (terms below 2^-126, fewer than 2^31 of them).  The
// rounds only take x and the branch from the sums as they are; the bounds are
// checked once per token by finish_f.  A wrong branch or run cannot pass: x
// then lies outside the segment, or within the bound of its edge.
// (The bounds themselves are in lda_internal.h, kEps and draw_tau on.)
constexpr uint16_t kDrawX = 0xFFFD;  // undecided: exact_draw
constexpr uint16_t kDrawM = 0xFFFC;  // in the max-topic branch, not checked yet
// Documents longer than this may hold a count that is not exact as the f16
// bits of fma_mix (an integer below 2^11 in the low half of an entry reads as
// that integer times 2^-24, subnormal or not); their tokens take draw_long_f.
constexpr uint32_t kMixCount = 2047;

struct WordF {
  const float *wf;
  const double *qb;
  int nb, K, qhalf;
  uint32_t K1;
  double a1, qp, alpha;
};

typedef const __attribute__((address_space(3))) float lds_f32;
__device__ __forceinline__ float wf_of(const float *__restrict__ wf, uint32_t e) {
  uint32_t a;
  asm("v_mad_u32_u16 %0, %1, 4, %2 op_sel:[1,0,0,0]"
      : "=v"(a)
      : "v"(e), "s"(uint32_t(reinterpret_cast<uintptr_t>(wf))));
  return *(lds_f32 *)(size_t)a;
}
// s + count(e) * W^': the count is the entry's low half read as f16, exact
// times 2^-24 for counts up to kMixCount.
__device__ __forceinline__ float fma_count(uint32_t e, float w, float s) {
  asm("v_fma_mix_f32 %0, %1, %2, %0 op_sel:[0,0,0] op_sel_hi:[1,0,0]" : "+v"(s) : "v"(e), "v"(w));
  return s;
}
// This lane's S' terms over a run of kRun entries: Mix for counts up to
// kMixCount, else any count.
template <bool Mix>
__device__ __forceinline__ double run_sum_f(const uint32_t (&r)[kRun], const float *__restrict__ wf) {
  float s = 0.0f;
#pragma unroll
  for (int i = 0; i < kRun; ++i) {
    if (Mix) s = fma_count(r[i], wf_of(wf, r[i]), s);
    else s = __builtin_fmaf(float(r[i] & 0xFFFFu), wf_of(wf, r[i]), s);
  }
  return Mix ? double(s) : double(s) * (1.0 / kWScale);
}
// What a round leaves of a token for finish_f: S' in bt.nnz (as a float) and,
// in bt.u, M - x for a draw in M, x inside the run for S' (the run in bt.off),
// x past M + S' for Q'.

// One round of small-group draws, as draw_small.
template <int G, int NC>
__device__ void draw_small_f(const BatchLds &bt, int slot, int n, const WordF &w, const uint32_t *__restrict__ d_ent,
                             int li) {
  constexpr uint32_t kSpan = uint32_t(G) * kRun;
  if (slot < n) {
    const int src = bt.list[slot];
    const uint32_t nc = (bt.nnz[src] + 1u + kSpan - 1) / kSpan;  // slots: header + entries
    const uint32_t off0 = bt.off[src];
    const uint32_t *run = d_ent + off0 + uint32_t(li) * kRun;
    const double u = bt.u[src];
    uint32_t r[NC][kRun];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      if (uint32_t(c) < nc) load_run<kRun>(run + c * kSpan, 0, r[c]);
    }
    if (li == 0) r[0][0] = uint32_t(w.K) << 16;  // the row header
    double s[NC], T[NC];
    uint32_t c1 = 0xFFFFFFFFu;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      s[c] = 0.0;
      if (uint32_t(c) < nc) {
        c1 = run_count_of<kRun>(r[c], w.K1, c1);
        s[c] = run_sum_f<true>(r[c], w.wf);
      }
    }
    double S = 0.0;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      S += gsum<G>(s[c]);
      T[c] = S;
    }
    c1 = gmin_u32<G>(c1);
    const double Mm = w.a1 * (double(c1 <= 0xFFFFu ? c1 : 0u) + w.alpha);  // Eq. 7
    const double x = u * ((Mm + S) + w.qp);
    if (li == 0) bt.nnz[src] = __float_as_uint(float(S));
    if (x >= Mm && x < Mm + S) {
      int cs = 0;
      double base = Mm, sc = s[0];
#pragma unroll
      for (int c = 1; c < NC; ++c) {
        if (uint32_t(c) < nc && x >= Mm + T[c - 1]) {
          cs = c;
          base = Mm + T[c - 1];
          sc = s[c];
        }
      }
      const double incl = gscan<G>(sc, li);
      const int sel = pick_lane<G>(sc, incl, base, x, li);
      if (li == sel) {
        bt.off[src] = (off0 + uint32_t(cs) * kSpan + uint32_t(li) * kRun) | (cs == 0 && li == 0 ? 1u : 0u);
        bt.u[src] = x - (base + (incl - sc));
        bt.top[src] = kDrawS;
      }
    } else if (li == 0) {
      bt.u[src] = x < Mm ? Mm - x : x - (Mm + S);
      bt.top[src] = x < Mm ? kDrawM : kDrawQ;
    }
  }
}

template <int G, int MaxNC>
__device__ void draw_rounds_f(int from, int to, const int (&ends)[8], const BatchLds &bt, const WordF &w,
                              const uint32_t *__restrict__ d_ent) {
  constexpr uint32_t kSpan = uint32_t(G) * kRun;
  for (int base = from; base < to; base += kWave / G) {
    const int ln = lane_here(), g = ln / G, li = ln % G;
    const int last = min(base + kWave / G, to) - 1;
    uint32_t upper = kBucketEnd[7];
#pragma unroll
    for (int k = 6; k >= 0; --k) upper = last < ends[k] ? kBucketEnd[k] : upper;
    const uint32_t nc = (upper + kSpan - 1) / kSpan;
    const int slot = base + g;
    if (nc <= 1) {
      draw_small_f<G, 1>(bt, slot, to, w, d_ent, li);
    } else if (nc == 2) {
      draw_small_f<G, 2>(bt, slot, to, w, d_ent, li);
    } else if (nc == 3) {
      draw_small_f<G, 3>(bt, slot, to, w, d_ent, li);
    } else if (MaxNC <= 4 || nc == 4) {
      draw_small_f<G, 4>(bt, slot, to, w, d_ent, li);
    } else {
      if constexpr (MaxNC > 4) {
        if (nc <= 6) draw_small_f<G, 6>(bt, slot, to, w, d_ent, li);
        else draw_small_f<G, MaxNC>(bt, slot, to, w, d_ent, li);
      }
    }
  }
}

// Tokens with rows of more than 512 slots or documents of more than kMixCount
// tokens, four at a time, one per 16-lane group, as draw_long: the later
// tokens of a run of one word in one document draw from the first one's sums.
__device__ void draw_long_f(unsigned long long mask, unsigned long long foll, unsigned long long starts,
                            const BatchLds &bt, const WordF &w, const uint32_t *__restrict__ d_ent, int grp, int li) {
  mask &= ~foll;  // the runs' first tokens
  while (mask) {
    const unsigned long long m1 = mask & (mask - 1ull), m2 = m1 & (m1 - 1ull), m3 = m2 & (m2 - 1ull);
    const int f0 = __ffsll((long long)mask) - 1, f1 = __ffsll((long long)m1) - 1;
    const int f2 = __ffsll((long long)m2) - 1, f3 = __ffsll((long long)m3) - 1;
    mask = m3 & (m3 - 1ull);
    const int src = grp == 0 ? f0 : grp == 1 ? f1 : grp == 2 ? f2 : f3;
    if (src >= 0) {
      const uint32_t off0 = bt.off[src];
      const uint32_t *row = d_ent + off0;  // slot 0 is the row header
      const uint32_t pad = uint32_t(w.K) << 16;
      const uint32_t slots = d_row_slots(bt.nnz[src]), nch = (slots + kChunk - 1) / kChunk;
      // the row's chunks, two loaded together; lane c of the group keeps the
      // total of the c-th m chunks, so that a draw walks only those m again
      const uint32_t m = (nch + uint32_t(kGroup) - 1u) / uint32_t(kGroup);
      uint32_t r[kRun], r2[kRun];
      double s = 0.0, incl = 0.0, S = 0.0, tot = 0.0;
      uint32_t c1 = 0xFFFFFFFFu, sup = 0, in_sup = 0;
      auto chunk = [&](const uint32_t (&rc)[kRun]) {
        c1 = run_count_of<kRun>(rc, w.K1, c1);
        s = run_sum_f<false>(rc, w.wf);
        incl = row_incl_scan(s);
        const double tch = __shfl(incl, kGroup - 1, kGroup);
        S += tch;
        tot += uint32_t(li) == sup ? tch : 0.0;
        if (++in_sup == m) {
          in_sup = 0;
          ++sup;
        }
      };
      if (nch == 1) {
        load_run_masked(row, 0, slots, li, pad, r);
        chunk(r);
      } else {
        // a row of several chunks: its slots are whole chunks, or 64 past one
        for (uint32_t ch = 0; ch < nch; ch += 2) {
          load_run_masked(row, ch, slots, li, pad, r);
          if (ch + 1 < nch) {
            load_run_masked(row, ch + 1, slots, li, pad, r2);
            chunk(r);
            chunk(r2);
          } else {
            chunk(r);
          }
        }
      }
      const double Mm = w.a1 * (double(row_sum_u32(c1 <= 0xFFFFu ? c1 : 0u)) + w.alpha);
      double mine = Mm;  // lane c's base: M and the totals before it, left to right
      {
        double cb = Mm;
        for (uint32_t c = 0; c * m < nch; ++c) {
          mine = uint32_t(li) == c ? cb : mine;
          cb += __shfl(tot, int(c), kGroup);
        }
      }
      const double Z = (Mm + S) + w.qp;
      auto draw = [&](int tok) {
        const double x = bt.u[tok] * Z;
        uint16_t code = x < Mm ? kDrawM : kDrawQ;
        if (x >= Mm && x < Mm + S) {
          code = kDrawX;
          uint32_t cs = 0;
          double base = Mm;
          bool found = nch == 1;
          if (nch > 1) {
            const uint32_t hm = uint32_t(__ballot(uint32_t(li) * m < nch && x < mine + tot) >> (grp * kGroup)) & kGroupMask;
            const uint32_t sel = hm ? uint32_t(__ffs(hm) - 1) : uint32_t(kGroup);
            base = __shfl(mine, int(sel & (kGroup - 1)), kGroup);
            const uint32_t to = hm ? min(nch, (sel + 1u) * m) : 0u;
            for (uint32_t ch = sel * m; ch < to && !found; ++ch) {
              load_run_masked(row, ch, slots, li, pad, r);
              s = run_sum_f<false>(r, w.wf);
              incl = row_incl_scan(s);
              const double total = __shfl(incl, kGroup - 1, kGroup);
              found = x < base + total;
              if (found) cs = ch;
              else base += total;
            }
          }
          if (found) {
            const int sel = run_lane(s, incl, base, x, grp);
            if (li == sel) {
              bt.off[tok] = (off0 + cs * kChunk + uint32_t(li) * kRun) | (cs == 0u && li == 0 ? 1u : 0u);
              bt.u[tok] = x - (base + (incl - s));
            }
            code = kDrawS;
          }
        }
        if (li == 0) {
          if (code == kDrawM || code == kDrawQ) bt.u[tok] = x < Mm ? Mm - x : x - (Mm + S);
          bt.nnz[tok] = __float_as_uint(float(S));
          bt.top[tok] = code;
        }
      };
      draw(src);
      // the run's later tokens: lanes after src up to the next run start
      const unsigned long long after = ~((2ull << src) - 1ull);  // the lanes above src
      const unsigned long long nxt = starts & after;
      unsigned long long fl = foll & after & (nxt ? (nxt & (0ull - nxt)) - 1ull : ~0ull);
      for (; fl; fl &= fl - 1ull) draw(__ffsll((long long)fl) - 1);
    }
  }
}

// The block of the Q' prefix that holds xq: the largest with qb[block] <= xq,
// for qb[0] <= xq < qb[nb].
__device__ __forceinline__ int q_block_f(const WordF &w, double xq) {
  int lo = 0;
  for (int step = w.qhalf; step > 0; step >>= 1) {
    const int at = min(lo + step, w.nb);
    lo = w.qb[at] <= xq ? at : lo;
  }
  return lo;
}

// The drawn topic of a batch token, one lane per token, or kDrawX where an
// edge of the segment lies within the bound.
template <int BS>
__device__ __forceinline__ uint32_t finish_f(int q, const BatchLds &bt, const WordF &w,
                                             const uint32_t *__restrict__ d_ent, uint32_t len) {
  const uint32_t code = bt.top[q];
  if (code == kDrawX) return kDrawX;
  const double xs = bt.u[q];
  const double S = double(__uint_as_float(bt.nnz[q])) * (1.0 + 0x1p-20);  // rounded up
  const double tau = draw_tau(w.a1 * (double(len) + w.alpha), S, w.qp);  // C1 <= len
  const double e2 = s_bound(S, tau);
  if (code == kDrawM) return xs > e2 ? uint32_t(kDrawM) : uint32_t(kDrawX);
  if (code == kDrawS) {
    const uint32_t a = bt.off[q];
    uint32_t r[kRun];
    load_run<kRun>(d_ent + (a & ~uint32_t(kRun - 1)), 0, r);
    if (a & 1u) r[0] = uint32_t(w.K) << 16;  // the run starts with the row header
    double p = 0.0, below = -1.0;
    uint32_t ent = 0;
#pragma unroll
    for (int i = 0; i < kRun; ++i) {
      const bool open = p <= xs;
      ent = open ? r[i] : ent;
      below = open ? p : below;
      p = __builtin_fma(double(r[i] & 0xFFFFu), double(wf_of(w.wf, r[i])) * (1.0 / kWScale), p);
    }
    // the chosen entry's edges
    const double above = __builtin_fma(double(ent & 0xFFFFu), double(wf_of(w.wf, ent)) * (1.0 / kWScale), below);
    return xs - below > e2 && above - xs > e2 && below >= 0.0 ? ent >> 16 : uint32_t(kDrawX);
  }
  if (!(xs < w.qb[w.nb]) || !(xs >= 0.0)) return kDrawX;
  const double eq1 = q_bound(S, w.qp, tau);
  const int lo = q_block_f(w, xs);
  // inside the block in fp32, in units of alpha * 2^-24
  const float inv = float(kWScale / w.alpha);
  const float xb = float((xs - w.qb[lo]) * (kWScale / w.alpha));
  const float *wb = w.wf + lo * BS;
  float p = 0.0f, below = 0.0f;
  int at = 0;
#pragma unroll 8
  for (int i = 0; i < BS; ++i) {
    const bool open = p <= xb;
    at = open ? i : at;
    below = open ? p : below;
    p += wb[i];
  }
  const float above = below + wb[at];
  const float eq = q_bound_f(eq1, inv, p, xb, BS);
  return xb - below > eq && above - xb > eq ? uint32_t(lo * BS + at) : uint32_t(kDrawX);
}

// One token by a whole wave, all in fp64: W^' of a topic is recomputed from
// its count (a dense row's own; a sparse row's from the single-precision
// value, whose rounding, 2^-24 of a count below 2^16 plus beta, leaves the
// integer, or by a search of the row when beta is large).
struct ExactRow {
  const int32_t *dense;   // the word's dense row, or null
  const uint32_t *ents;   // its sparse row otherwise
  uint32_t nnz;
};
__device__ double exact_w(const DevState &d, const Params &p, const WordF &w, const ExactRow &er, uint32_t k) {
  if (k >= uint32_t(w.K) || k == w.K1) return 0.0;
  const double den = d.den[k];
  if (er.dense) return what(uint32_t(er.dense[k]), p.beta, den);
  if (p.beta <= 1e6) return (rint(double(w.wf[k]) * (1.0 / kWScale) * den - p.beta) + p.beta) / den;
  const uint32_t lb = row_lower_bound(er.ents, er.nnz, k);
  return what(lb < er.nnz && (er.ents[lb] >> 16) == k ? er.ents[lb] & 0xFFFFu : 0u, p.beta, den);
}
// Returns the topic, bit 16 set for a draw in the max-topic branch.
constexpr uint32_t kExactM = 0x10000u;
template <int BS>
__device__ uint32_t exact_draw(const DevState &d, const Params &p, const WordF &w, const ExactRow &er, uint32_t off,
                               double u, int lane) {
  const uint32_t *row = d.d_ent + off;
  const uint32_t nnz = __builtin_amdgcn_readfirstlane(row[0]) & 0xFFFFu;
  double S = 0.0;
  uint32_t C1 = 0;
  double term = 0.0;
  uint32_t k = 0;
  auto load = [&](uint32_t q0) {
    const uint32_t q = q0 + uint32_t(lane);
    const uint32_t ent = q < nnz ? row[1u + q] : uint32_t(w.K) << 16;
    k = ent >> 16;
    term = double(ent & 0xFFFFu) * exact_w(d, p, w, er, k);
    return ent;
  };
  for (uint32_t q0 = 0; q0 < nnz; q0 += kWave) {
    const uint32_t ent = load(q0);
    S += __shfl(wave_incl_scan(term), kWave - 1);
    const unsigned long long m = __ballot((ent >> 16) == w.K1);
    if (m) C1 = max(C1, uint32_t(__shfl(int(ent & 0xFFFFu), __ffsll((long long)m) - 1)));
  }
  const double Mm = w.a1 * (double(C1) + w.alpha);
  const double x = u * ((Mm + S) + w.qp);
  if (x < Mm) return w.K1 | kExactM;
  uint32_t last = w.K1;  // the last segment of positive width
  if (x < Mm + S) {
    double base = Mm;
    for (uint32_t q0 = 0; q0 < nnz; q0 += kWave) {
      load(q0);
      const double incl = wave_incl_scan(term);
      const unsigned long long pos = __ballot(term > 0.0), hit = __ballot(term > 0.0 && x < base + incl);
      if (hit) return uint32_t(__shfl(int(k), __ffsll((long long)hit) - 1));
      if (pos) last = uint32_t(__shfl(int(k), 63 - __clzll((long long)pos)));
      base += __shfl(incl, kWave - 1);
    }
    return last;
  }
  const double xq = x - (Mm + S);
  if (!(xq < w.qb[w.nb])) return (w.K1 == uint32_t(w.K - 1)) ? uint32_t(w.K - 2) : uint32_t(w.K - 1);
  const int lo = q_block_f(w, xq);
  k = uint32_t(lo * BS + lane);
  term = lane < BS ? w.alpha * exact_w(d, p, w, er, k) : 0.0;
  const double incl = w.qb[lo] + wave_incl_scan(term);
  const unsigned long long pos = __ballot(term > 0.0), hit = __ballot(term > 0.0 && xq < incl);
  if (hit) return uint32_t(__shfl(int(k), __ffsll((long long)hit) - 1));
  return pos ? uint32_t(__shfl(int(k), 63 - __clzll((long long)pos))) : last;
}

// Entries of the single-precision row: K + 1 rounded up to whole waves.
__host__ __device__ inline int wf_entries(int K) { return (K + kWave) / kWave * kWave; }

// Per iteration: qbase[b] = sum of alpha * beta/den[k] over block b of BS
// topics, what a word's Q' prefix starts from.
template <int BS>
__global__ __launch_bounds__(kBlock) void k_block_base(DevState d, Params p) {
  const int k = int(blockIdx.x) * kBlock + int(threadIdx.x);
  double v = k < p.K ? p.alpha * d.bden[k] : 0.0;
  v = group_sum<BS>(v);
  if (k % BS == 0 && k < p.K) d.qbase[k / BS] = v;
}

// The sampler of the units, NB threads per workgroup: as k_sampler, with
// the single-precision row.  A unit's setup touches only what changes: after
// another sparse word the previous word's topics go back to beta/den[k], the
// new word's entries are written and their excess over beta/den[k] is added
// to their blocks, then the K / BS block sums are scanned.  exact_draw compares
// with these sums, so they are whole numbers (q_units): their bits depend on
// the counts alone, not on the waves' timing, the cut or whether the row is
// dense (fp64 atomics took as long: 8.64 ms a launch for 20M tokens at
// K = 32,768, whole numbers 8.65).  At K = 32,768 the two-tile fp64 sampler
// filled three tiles of 16,400 topics per region.
template <int NB>
__device__ __forceinline__ void sampler_f_body(DevState d, Params p, uint32_t t,
                                               unsigned long long *__restrict__ stats) {
  extern __shared__ double lds[];
  constexpr int BS = q_block_topics(NB);
  const int K = p.K;
  const int nb = (K + BS - 1) / BS;
  const int nwf = wf_entries(K);
  const bool by_doc = doc_marks(d, p, t);
  float *wf = reinterpret_cast<float *>(lds);                        // [nwf]
  double *qb = lds + nwf / 2;                                        // [nb + 1]
  double *s_u = qb + nb + 1;                                        // [NB]
  uint32_t *s_off = reinterpret_cast<uint32_t *>(s_u + NB);          // [NB]
  uint32_t *s_nnz = s_off + NB;                                      // [NB]
  uint32_t *s_reg = s_nnz + NB;                                      // [4]
  uint16_t *s_top = reinterpret_cast<uint16_t *>(s_reg + 4);         // [NB]
  uint8_t *s_list = reinterpret_cast<uint8_t *>(s_top + NB);         // [NB]
  const int qhalf = q_blocks_padded(nb + 1) / 2;  // the first step of a search over qb[0..nb]
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  if (blockIdx.x == 0 && tid == 0) stats[ST_MARKS] = by_doc ? 2ull : 1ull;
  const BatchLds bt{s_off + wave * kWave, s_nnz + wave * kWave, s_u + wave * kWave, s_top + wave * kWave, nullptr,
                    s_list + wave * kWave};
  for (int k = K + tid; k < nwf; k += NB) wf[k] = 0.0f;
  uint32_t cur = 0xFFFFFFFFu, K1 = 0;
  double a1 = 0.0, qp = 0.0;
  unsigned long long *qi = reinterpret_cast<unsigned long long *>(qb);  // the block sums before the prefix is taken
  const int32_t *wrow = nullptr;   // the word's dense row, or null
  const uint32_t *held = nullptr;  // the sparse word whose row wf holds
  uint32_t held_nnz = 0, held_k1 = 0;
  // (tokens of a corpus, and so these counts, fit 32 bits)
  uint32_t n_sampled = 0, n_after_s = 0, n_reg = 0, n_dreg = 0;
  unsigned long long nnz_sum = 0, row_bytes = 0;

  for (;;) {
    if (tid == 0) {
      const int64_t r = int64_t(atomicAdd(&d.counters[CNT_SAMPLER], 1u));
      s_reg[3] = r < p.n_units ? 1u : 0u;
      if (s_reg[3]) {
        s_reg[0] = d.unit[3 * size_t(r)];
        s_reg[1] = d.unit[3 * size_t(r) + 1];
        s_reg[2] = d.unit[3 * size_t(r) + 2];
      }
    }
    __syncthreads();
    if (!s_reg[3]) break;
    const uint32_t vc = __builtin_amdgcn_readfirstlane(s_reg[0]), v = vc & ~kUnitContinues;
    const uint32_t b = __builtin_amdgcn_readfirstlane(s_reg[1]);
    const uint32_t e = __builtin_amdgcn_readfirstlane(s_reg[2]);
    if (vc == v) {  // the first unit of its region
      n_reg++;
      if (int32_t(v) < p.n_dense) n_dreg++;
    }
    if (b == d.word_off[v])
      row_bytes += int32_t(v) < p.n_dense ? 4ull * uint64_t(K) : 4ull * d.ws_nnz[int(v) - p.n_dense];
    if (v != cur) {
      cur = v;
      const WordRec rec = d.wrec[v];
      K1 = rec.k1;
      a1 = rec.a1;
      qp = rec.qp;
      const int ex = q_exponent(qp);
      // every block starts from the topics that the word does not hold; K1's
      // from its other topics, by the last wave (the one with the fewest
      // entries), the load ahead of the rest
      const int b1 = int(K1) / BS, kb = b1 * BS + lane;
      const bool lw = wave == NB / kWave - 1;
      double others = lw && lane < BS && kb < K && uint32_t(kb) != K1 ? d.bden[kb] : 0.0;
      for (int q = tid; q < nb; q += NB) qi[q + 1] = q == b1 ? 0ull : q_units(d.qbase[q], ex);
      auto add_others = [&]() {
        if (lw) {
          others = wave_incl_scan(p.alpha * others);
          if (lane == BS - 1 && b1 < nb) atomicAdd(&qi[b1 + 1], q_units(others, ex));
        }
      };
      if (int32_t(v) < p.n_dense) {
        wrow = d.w_dense + size_t(v) * size_t(K);
        __syncthreads();
        for (int k0 = wave * kWave; k0 < K; k0 += NB) {
          const int k = k0 + lane;
          const bool in = k < K && uint32_t(k) != K1;
          const double w = in ? what(uint32_t(wrow[k]), p.beta, d.den[k]) : 0.0;
          wf[k] = float(w * kWScale);
          // (a topic that the word does not hold adds nothing)
          const unsigned long long sum = row_incl_scan_u64(in ? q_units(p.alpha * (w - d.bden[k]), ex) : 0ull);
          if (lane % kGroup == kGroup - 1 && sum) atomicAdd(&qi[k / BS + 1], sum);
        }
        add_others();
        held = nullptr;
        __syncthreads();
      } else {
        const int s = int(v) - p.n_dense;
        const uint32_t *ents = d.ws_ent + d.ws_cap[s];
        const uint32_t nnz = d.ws_nnz[s];
        wrow = nullptr;
        if (held) {
          for (uint32_t q = tid; q < held_nnz; q += NB) {
            const uint32_t k = held[q] >> 16;
            wf[k] = float(d.bden[k] * kWScale);
          }
          if (tid == 0 && held_k1 < uint32_t(K)) wf[held_k1] = float(d.bden[held_k1] * kWScale);  // K1 = K in two-branch mode
        } else {
          for (int k = tid; k < K; k += NB) wf[k] = float(d.bden[k] * kWScale);
        }
        __syncthreads();
        for (uint32_t q = tid; q < nnz; q += NB) {
          const uint32_t ent = ents[q], k = ent >> 16;
          const double w = what(ent & 0xFFFFu, p.beta, d.den[k]);
          wf[k] = float(w * kWScale);
          if (k != K1) atomicAdd(&qi[k / BS + 1], q_units(p.alpha * (w - d.bden[k]), ex));
        }
        add_others();
        held = ents;
        held_nnz = nnz;
        held_k1 = K1;
        __syncthreads();
        if (tid == 0) wf[K1] = 0.0f;  // the max topic is its own branch (Eq. 5)
      }
      // the prefix over the blocks: a scan per wave, then the totals of the
      // waves before, in round and wave order
      double *s_tot = s_u;  // [rounds * waves <= NB]; s_u is next written by the token batches
      for (int r = 0; r * NB < nb; ++r) {
        const int blk = r * NB + tid;
        const double incl = wave_incl_scan(blk < nb ? q_value(qi[blk + 1], ex) : 0.0);
        if (blk < nb) qb[blk + 1] = incl;
        if (lane == kWave - 1) s_tot[r * (NB / kWave) + wave] = incl;
      }
      __syncthreads();
      {
        double acc = 0.0;
        for (int r = 0; r * NB < nb; ++r) {
          double own = 0.0;
          for (int w = 0; w < NB / kWave; ++w) {
            if (w == wave) own = acc;
            acc += s_tot[r * (NB / kWave) + w];
          }
          const int blk = r * NB + tid;
          if (blk < nb) qb[blk + 1] = own + qb[blk + 1];
        }
        if (tid == 0) qb[0] = 0.0;
      }
      __syncthreads();
    }

    const WordF w{wf, qb, nb, K, qhalf, K1, a1, qp, p.alpha};
    const uint32_t bsz = min(uint32_t(kWave), max(16u, ((e - b + uint32_t(NB / kWave) - 1u) / uint32_t(NB / kWave) + 15u) & ~15u));
    for (uint32_t base = b + uint32_t(wave) * bsz; base < e; base += uint32_t(NB / kWave) * bsz) {
      const int ln = lane_here();
      const uint32_t j = base + uint32_t(ln);
      const uint32_t be = min(e, base + bsz);
      uint32_t sk = 0, key = 0, off = 0;
      if (j < be) {
        const uint2 kr = d.wt_kr[j];
        key = kr.x;
        off = kr.y;
        sk = by_doc ? d.skip_doc[key >> 5] >> (key & 31u) : d.skip_bits[j >> 5] >> (j & 31u);
      }
      const bool und = j < be && !(sk & 1u);
      uint32_t hdr = 0;
      if (und) {
        hdr = d.d_ent[off];
        bt.off[ln] = off;
        bt.nnz[ln] = hdr & 0xFFFFu;
        bt.u[ln] = uniform_draw(p.seed, t, key);
      }
      const uint32_t nnz = hdr & 0xFFFFu;
      // long rows, and documents whose counts may pass fma_mix
      const bool lng = und && (nnz + 1u > 512u || (hdr >> 16) > kMixCount);
      const unsigned long long lmask = __ballot(lng);
      unsigned long long starts = 0ull;
      bool fol = false;
      if (lmask) {
        const uint32_t prev_off = uint32_t(__shfl(int(off), ln - 1));
        starts = __ballot(ln == 0 || off != prev_off);
        const unsigned long long below = ln ? ~0ull >> (64 - ln) : 0ull;
        const int rs = 63 - __clzll((long long)(starts & (below | (1ull << ln))));  // this lane's run start
        fol = lng && (lmask & below & (~0ull << rs)) != 0ull;
      }
      n_sampled += uint32_t(__popcll(__ballot(und)));
      nnz_sum += wave_sum_u32(fol && nnz + 1u > 512u ? min(nnz, uint32_t(kChunk)) : nnz);
      // the other rows by length bucket: groups of 4, 8 or 16 lanes
      const bool sml = und && !lng;
      int n = 0, ends[8];
      const uint32_t slots = nnz + 1u;
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const uint32_t lo = k ? kBucketEnd[k - 1] : 0u;
        const unsigned long long m = __ballot(sml && slots > lo && slots <= kBucketEnd[k]);
        if ((m >> ln) & 1ull)
          bt.list[n + int(__builtin_amdgcn_mbcnt_hi(uint32_t(m >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(m), 0u)))] =
              uint8_t(ln);
        n += __popcll(m);
        ends[k] = n;
      }
      const int left = ends[3] % 16;
      const int a = left > 0 && left <= 8 && ends[3] - ends[2] >= left ? ends[3] - left : ends[3];
      draw_rounds_f<4, 4>(0, a, ends, bt, w, d.d_ent);
      if (NB >= 1024) {
        draw_rounds_f<8, 8>(a, ends[7], ends, bt, w, d.d_ent);
      } else {
        draw_rounds_f<8, 4>(a, ends[5], ends, bt, w, d.d_ent);
        draw_rounds_f<16, 4>(ends[5], ends[7], ends, bt, w, d.d_ent);
      }
      if (lmask) draw_long_f(lmask, __ballot(fol), starts, bt, w, d.d_ent, ln / kGroup, ln % kGroup);
      uint32_t topic = K1;
      if (und) topic = finish_f<BS>(ln, bt, w, d.d_ent, hdr >> 16);
      n_after_s += uint32_t(__popcll(__ballot(topic == uint32_t(kDrawM))));
      topic = topic == uint32_t(kDrawM) ? K1 : topic;
      // the undecided tokens, by the whole wave in fp64
      for (unsigned long long m = __ballot(und && topic == uint32_t(kDrawX)); m; m &= m - 1ull) {
        const int q = __ffsll((long long)m) - 1;
        const uint32_t q_off = __builtin_amdgcn_readlane(off, q), q_key = __builtin_amdgcn_readlane(key, q);
        const uint32_t k = __builtin_amdgcn_readfirstlane(
            exact_draw<BS>(d, p, w, ExactRow{wrow, held, held_nnz}, q_off, uniform_draw(p.seed, t, q_key), ln));
        n_after_s += k >> 16;
        if (ln == q) topic = k & 0xFFFFu;
      }
      if (j < be) d.z_w[j] = uint16_t(topic);
    }
    __syncthreads();
  }
  if (lane == 0)
    store_stats(d, blockIdx.x * uint32_t(NB / kWave) + uint32_t(wave), wave == 0, n_sampled, n_after_s, nnz_sum, n_reg,
                n_dreg, row_bytes);
}
__global__ __launch_bounds__(256, 7) void k_sampler_f(DevState d, Params p, uint32_t t,
                                                      unsigned long long *__restrict__ stats) {
  sampler_f_body<256>(d, p, t, stats);
}
__global__ __launch_bounds__(512, 6) void k_sampler_f_512(DevState d, Params p, uint32_t t,
                                                          unsigned long long *__restrict__ stats) {
  sampler_f_body<512>(d, p, t, stats);
}
__global__ __launch_bounds__(1024, 4) void k_sampler_f_1024(DevState d, Params p, uint32_t t,
                                                            unsigned long long *__restrict__ stats) {
  sampler_f_body<1024>(d, p, t, stats);
}

// One statistic (0..kFoldBlocks-1) over the slots of the waves that stored
// it, by one workgroup of kBlock threads; added, since an out-of-core
// iteration folds once per chunk.
__device__ void fold_stat(const DevState &d, const StatSlots &sl, int which) {
  __shared__ unsigned long long red[kBlock / kWave];
  const bool skip = which == kFoldBlocks - 1;
  const unsigned long long *st = d.wave_stats + size_t(which) * kWaveSlots;
  unsigned long long s = 0;
  auto add = [&](int slot0, int n) {
#pragma unroll 4
    for (int q = int(threadIdx.x); q < n; q += kBlock) s += st[slot0 + q];
  };
  if (skip) {
    add(0, sl.doc);
  } else {
    add(0, sl.main);
    add(sl.light0, sl.light);
  }
  s = group_sum_u64<kWave>(s);
  if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x / kWave] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int q = 1; q < kBlock / kWave; ++q) s += red[q];
    constexpr int to[kFoldBlocks] = {ST_SAMPLED, ST_SKIP_AFTER_S, ST_NNZ, ST_REGIONS, ST_DENSE_REGIONS, ST_ROW_BYTES,
                                     ST_SKIP3};
    d.stats[to[which]] += s;
    if (skip) d.skip_hist[sl.t & 1u] += s;
  }
}
__global__ __launch_bounds__(kBlock) void k_fold_stats(DevState d, StatSlots sl) { fold_stat(d, sl, int(blockIdx.x)); }

// Rows of split dense words are accumulated with atomics; clear them and T.
// fold: the first kFoldBlocks workgroups also add up the iteration's statistics.
__global__ __launch_bounds__(kBlock) void k_zero_split(DevState d, Params p, StatSlots sl, int fold) {
  if (fold && blockIdx.x < kFoldBlocks) fold_stat(d, sl, int(blockIdx.x));
  const int64_t total = int64_t(p.n_dense) * p.K;
  for (int64_t x = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; x < total; x += int64_t(gridDim.x) * blockDim.x) {
    if (d.split[x / p.K]) d.w_dense[x] = 0;
  }
  for (int64_t k = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; k < p.K; k += int64_t(gridDim.x) * blockDim.x)
    d.T[k] = 0u;
}

constexpr int kHistAhead = 8;  // word-ordered topic loads per thread issued together in the W rebuild

// W rebuild (Sec. 4.3) for K below kWBitsK by one wave per region, the regions dealt
// round-robin over the waves of the grid, with no workgroup barrier per
// region: the region's counts in the wave's LDS table, then the dense row
// written whole (added with atomics when the word is split) or the sparse
// row compacted in ascending topic order, 64 topics per step by ballot; the
// table is cleared as it is read.  T is accumulated per workgroup in LDS and
// added to the device once at the end.
__global__ __launch_bounds__(kBlock) void k_rebuild_w_wave(DevState d, Params p) {
  extern __shared__ uint32_t ldsu[];
  const int K = p.K;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave, tid = threadIdx.x;
  uint32_t *tloc = ldsu;                                  // [K], the workgroup's
  uint32_t *hist = ldsu + size_t(K) * size_t(1 + wave);  // [K], the wave's
  for (int k = tid; k < K; k += kBlock) tloc[k] = 0u;
  for (int k = lane; k < K; k += kWave) hist[k] = 0u;
  __syncthreads();
  uint32_t bad = 0;
  const int64_t nwaves = int64_t(gridDim.x) * (kBlock / kWave);
  for (int64_t r = int64_t(blockIdx.x) * (kBlock / kWave) + wave; r < p.n_regions; r += nwaves) {
    const uint32_t v = d.region[3 * size_t(r)], b = d.region[3 * size_t(r) + 1], e = d.region[3 * size_t(r) + 2];
    for (uint32_t j0 = b + uint32_t(lane); j0 < e; j0 += uint32_t(kHistAhead * kWave)) {
      uint32_t zz[kHistAhead];
#pragma unroll
      for (int u = 0; u < kHistAhead; ++u) zz[u] = uint32_t(u * kWave) < e - j0 ? uint32_t(d.z_w[j0 + u * kWave]) : 0u;
#pragma unroll
      for (int u = 0; u < kHistAhead; ++u) {
        if (uint32_t(u * kWave) < e - j0) {
          if (zz[u] < uint32_t(K)) atomicAdd(&hist[zz[u]], 1u);
          else bad++;
        }
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // a wave's LDS accesses run in order
    if (int32_t(v) < p.n_dense) {
      int32_t *wrow = d.w_dense + size_t(v) * size_t(K);
      const bool split = d.split[v] != 0;
      for (int k = lane; k < K; k += kWave) {
        const uint32_t h = hist[k];
        hist[k] = 0u;
        if (h) atomicAdd(&tloc[k], h);
        if (!split) wrow[k] = int32_t(h);
        else if (h) atomicAdd(&wrow[k], int32_t(h));
      }
    } else {
      const int s = int(v) - p.n_dense;
      uint32_t *out = d.ws_ent + d.ws_cap[s];
      uint32_t base = 0;
      for (int k0 = 0; k0 < K; k0 += kWave) {
        const int k = k0 + lane;
        uint32_t h = 0;
        if (k < K) {
          h = hist[k];
          hist[k] = 0u;
        }
        const unsigned long long m = __ballot(h != 0u);
        if (h) {
          atomicAdd(&tloc[k], h);
          const uint32_t rank = __builtin_amdgcn_mbcnt_hi(uint32_t(m >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(m), 0u));
          out[base + rank] = (uint32_t(k) << 16) | h;
        }
        base += uint32_t(__popcll(m));
      }
      if (lane == 0) d.ws_nnz[s] = base;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  }
  __syncthreads();
  for (int k = tid; k < K; k += kBlock)
    if (tloc[k]) atomicAdd(&d.T[k], tloc[k]);
  if (bad) atomicAdd(&d.stats[ST_ERRORS], (unsigned long long)bad);
}

// W rebuild for K >= kWBitsK: the touched topics of a region are marked in
// a bitmap, so the work per region follows its tokens, not K.
// Packed: two 16-bit counts per LDS word (every region shorter than 2^16
// tokens), which halves the table (two workgroups per CU at K = 32,768).
// T is left to k_topic_hist and k_topic_reduce: adding each region's counts
// into T with device atomics cost more than the rest of the rebuild.
template <bool Packed>
__global__ __launch_bounds__(kBlock) void k_rebuild_w_bits(DevState d, Params p) {
  extern __shared__ uint32_t ldsu[];
  const int K = p.K;
  const int nw = (K + 31) / 32;
  const int nh = Packed ? (K + 1) / 2 : K;
  uint32_t *hist = ldsu;                              // [nh]: the region's topic counts
  uint32_t *bits = ldsu + nh;                         // [nw]: topics with a nonzero count
  __shared__ uint32_t s_scan[kBlock / kWave];
  const int tid = threadIdx.x;
  uint32_t bad = 0;
  auto count = [&](int k) -> uint32_t { return Packed ? (hist[k >> 1] >> ((k & 1) << 4)) & 0xFFFFu : hist[k]; };
  for (int k = tid; k < nh; k += kBlock) hist[k] = 0u;
  for (int q = tid; q < nw; q += kBlock) bits[q] = 0u;
  __syncthreads();
  // regions dealt round-robin over the workgroups
  for (int64_t r = blockIdx.x; r < p.n_regions; r += gridDim.x) {
    const uint32_t v = d.region[3 * size_t(r)], b = d.region[3 * size_t(r) + 1], e = d.region[3 * size_t(r) + 2];
    // kHistAhead topic loads per thread in flight at once
    for (uint32_t j0 = b + tid; j0 < e; j0 += uint32_t(kHistAhead * kBlock)) {
      uint32_t zz[kHistAhead];
#pragma unroll
      for (int u = 0; u < kHistAhead; ++u) zz[u] = uint32_t(u * kBlock) < e - j0 ? uint32_t(d.z_w[j0 + u * kBlock]) : 0u;
#pragma unroll
      for (int u = 0; u < kHistAhead; ++u) {
        if (uint32_t(u * kBlock) < e - j0) {
          const uint32_t z = zz[u];
          if (z < uint32_t(K)) {
            if (Packed) atomicAdd(&hist[z >> 1], 1u << ((z & 1u) << 4));
            else atomicAdd(&hist[z], 1u);
            atomicOr(&bits[z >> 5], 1u << (z & 31u));
          } else {
            bad++;
          }
        }
      }
    }
    __syncthreads();
    // the touched topics, each thread a contiguous run of bitmap words (ascending)
    const int per = (nw + kBlock - 1) / kBlock;
    const int q0 = min(nw, tid * per), q1 = min(nw, q0 + per);
    if (int32_t(v) < p.n_dense) {
      int32_t *wrow = d.w_dense + size_t(v) * size_t(K);
      if (d.split[v]) {
        for (int q = q0; q < q1; ++q)
          for (uint32_t m = bits[q]; m; m &= m - 1u) {
            const int k = q * 32 + __ffs(m) - 1;
            atomicAdd(&wrow[k], int32_t(count(k)));
          }
      } else {
        for (int k = tid; k < K; k += kBlock) wrow[k] = int32_t(count(k));
      }
    } else {
      const int s = int(v) - p.n_dense;
      uint32_t cnt = 0;
      for (int q = q0; q < q1; ++q) cnt += uint32_t(__popc(bits[q]));
      uint32_t total = 0;
      uint32_t off = block_exclusive_u32(cnt, s_scan, &total);
      uint32_t *out = d.ws_ent + d.ws_cap[s];
      for (int q = q0; q < q1; ++q)
        for (uint32_t m = bits[q]; m; m &= m - 1u) {
          const int k = q * 32 + __ffs(m) - 1;
          out[off++] = (uint32_t(k) << 16) | count(k);
        }
      if (tid == 0) d.ws_nnz[s] = total;
    }
    __syncthreads();  // the non-split dense row reads every hist entry
    for (int q = q0; q < q1; ++q) {
      const uint32_t mq = bits[q];
      // cleared once both counts of a word are read (a word's two topics
      // are in the same bitmap word)
      for (uint32_t m = mq; m; m &= m - 1u) {
        const int k = q * 32 + __ffs(m) - 1;
        hist[Packed ? k >> 1 : k] = 0u;
      }
      bits[q] = 0u;
    }
    __syncthreads();
  }
  if (bad) atomicAdd(&d.stats[ST_ERRORS], (unsigned long long)bad);
}

// T for large K: the histogram of the word-ordered topics.  Each workgroup
// counts a slice of the tokens (8-token aligned, 8 topics a load) in LDS and
// writes its counts to its row of scratch; k_topic_reduce adds the rows into
// T (zeroed by k_zero_split, so out-of-core chunks add up).
constexpr int kHistBlock = 1024;
__global__ __launch_bounds__(kHistBlock) void k_topic_hist(DevState d, Params p, uint32_t *__restrict__ rows) {
  extern __shared__ uint32_t ldsu[];
  const int K = p.K;
  for (int k = threadIdx.x; k < K; k += kHistBlock) ldsu[k] = 0u;
  __syncthreads();
  const int64_t n = p.n, g = blockIdx.x, G = gridDim.x;
  const int64_t b = (n * g / G) & ~int64_t(7), e = g + 1 == G ? n : (n * (g + 1) / G) & ~int64_t(7);
  int64_t j = b + int64_t(threadIdx.x) * 8;
  for (; j + 8 <= e; j += int64_t(kHistBlock) * 8) {
    const uint4 v = *reinterpret_cast<const uint4 *>(d.z_w + j);
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t z0 = w[i] & 0xFFFFu, z1 = w[i] >> 16;
      if (z0 < uint32_t(K)) atomicAdd(&ldsu[z0], 1u);
      if (z1 < uint32_t(K)) atomicAdd(&ldsu[z1], 1u);
    }
  }
  for (; j < e; ++j) {  // the slice's last tokens past a whole 8 (at most 7, one thread)
    const uint32_t z = d.z_w[j];
    if (z < uint32_t(K)) atomicAdd(&ldsu[z], 1u);
  }
  __syncthreads();
  uint32_t *row = rows + size_t(g) * size_t(K);
  for (int k = threadIdx.x; k < K; k += kHistBlock) row[k] = ldsu[k];
}

__global__ __launch_bounds__(kBlock) void k_topic_reduce(DevState d, Params p, const uint32_t *__restrict__ rows,
                                                         int G) {
  const int k = int(blockIdx.x) * kBlock + int(threadIdx.x);
  if (k >= p.K) return;
  uint32_t s = 0;
  for (int g = 0; g < G; ++g) s += rows[size_t(g) * size_t(p.K) + size_t(k)];
  if (s) atomicAdd(&d.T[k], s);
}

constexpr int kPre = 2;   // chunks of 64 tokens per document gathered one document ahead
constexpr int kTail = 4;  // chunks of 64 tokens gathered together past the first kPre

// Inclusive prefix sum of a u32 over the 64 lanes of a wave: DPP shifts
// inside each row of 16 lanes (lanes below the shift read 0), then the row
// totals carried across rows.
__device__ __forceinline__ uint32_t wave_incl_scan_u32(uint32_t v, int lane) {
  v += uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x111, 0xF, 0xF, true));
  v += uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x112, 0xF, 0xF, true));
  v += uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x114, 0xF, 0xF, true));
  v += uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x118, 0xF, 0xF, true));
  const uint32_t r0 = __builtin_amdgcn_readlane(v, 15), r1 = __builtin_amdgcn_readlane(v, 31),
                 r2 = __builtin_amdgcn_readlane(v, 47);
  v += lane >= 16 ? r0 : 0u;
  v += lane >= 32 ? r1 : 0u;
  v += lane >= 48 ? r2 : 0u;
  return v;
}

// The D row of one document from its topic histogram (16-bit counts, two
// per word of hist) and the bitmap of its topics, by one wave: 64 bitmap
// words (2048 topics) per step, one per lane, each lane listing its word's
// topics at its prefix-sum offset, then one lane per listed topic writing the
// packed entry (topic << 16 | count) in ascending topic order.  The two
// topics of a count word share a bitmap word, so both are listed in the same
// step.  The table and the bitmap are left clear; out points at the row's
// first entry, the header (len << 16 | nnz) goes before it and the padding
// entries (topic K, count 0) after the entries.
__device__ __forceinline__ void emit_row(uint32_t *__restrict__ hist, uint32_t *__restrict__ bits, uint16_t *__restrict__ list, int nw,
                         int K, uint32_t *__restrict__ out, uint32_t len, int lane) {
  uint32_t base = 0;
  for (int q0 = 0; q0 < nw; q0 += kWave) {
    const int q = q0 + lane;
    uint32_t m = 0;
    if (q < nw) {
      m = bits[q];
      bits[q] = 0u;
    }
    const uint32_t cnt = uint32_t(__popc(m));
    const uint32_t incl = wave_incl_scan_u32(cnt, lane);
    const uint32_t n = __builtin_amdgcn_readlane(incl, kWave - 1);
    if (n == 0u) continue;
    uint32_t o = incl - cnt;
    while (m) {
      const uint32_t bit = uint32_t(__ffs(m) - 1);
      m &= m - 1u;
      list[o++] = uint16_t(uint32_t(q) * 32u + bit);
    }
    __threadfence_block();
    for (uint32_t j = uint32_t(lane); j < n; j += kWave) {
      const uint32_t z = list[j];
      const uint32_t zn = j + 1u < n ? uint32_t(list[j + 1u]) : 0xFFFFFFFFu;
      const uint32_t w = hist[z >> 1];
      out[base + j] = (z << 16) | ((z & 1u) ? (w >> 16) : (w & 0xFFFFu));
      // clear a count word after its last listed topic has been read
      if ((z & 1u) || zn != z + 1u) hist[z >> 1] = 0u;
    }
    __threadfence_block();
    base += n;
  }
  for (uint32_t q = base + uint32_t(lane); q + 1u < d_row_slots(base); q += kWave) out[q] = uint32_t(K) << 16;
  if (lane == 0) out[-1] = (len << 16) | base;
  __threadfence_block();
}

// The D rows of the heavy documents (longer than kHeavyDoc), one workgroup
// per document, before the workgroup's waves turn to the light documents.
// Each wave gathers topics of its share of the tokens through the inverted
// index into its own histogram and bitmap (so that LDS atomics contend only
// inside a wave), the tables are added into wave 0's (two 16-bit counts per
// word: a document's counts stay below 2^16, so the halves never carry), and
// wave 0 emits the row.  Every table is left clear.
__device__ void heavy_rebuild_d(const DevState &d, const Params &p, uint32_t *__restrict__ lds, uint32_t &bad) {
  __shared__ uint32_t s_next;
  const int K = p.K, half = (K + 1) / 2, nw = (K + 31) / 32;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), nthr = int(blockDim.x), waves = nthr / kWave;
  const size_t words = d_rebuild_lds_words(K);
  uint32_t *hist = lds + size_t(tid / kWave) * words;
  uint32_t *bits = hist + half;
  for (;;) {
    __syncthreads();  // the tables are clear, s_next is free
    if (tid == 0) s_next = atomicAdd(&d.counters[CNT_HEAVY_REBUILD], 1u);
    __syncthreads();
    const uint32_t h = s_next;
    if (h >= uint32_t(p.n_heavy)) break;
    const uint32_t dd = d.heavy_docs[h];
    const uint32_t b = d.doc_off[dd], e = d.doc_off[dd + 1];
    for (uint32_t p0 = b + uint32_t(tid); p0 < e; p0 += uint32_t(4 * nthr)) {
      uint32_t zz[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const uint32_t pp = p0 + uint32_t(c * nthr);
        zz[c] = pp < e ? d.dt_wpos[pp] : 0u;
      }
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (p0 + uint32_t(c * nthr) < e) zz[c] = d.z_w[zz[c]];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        if (p0 + uint32_t(c * nthr) < e) {
          const uint32_t z = zz[c];
          if (z < uint32_t(K)) {
            atomicAdd(&hist[z >> 1], (z & 1u) ? 0x10000u : 1u);
            atomicOr(&bits[z >> 5], 1u << (z & 31u));
          } else {
            bad++;
          }
        }
      }
    }
    __syncthreads();
    // the other waves' tables added into wave 0's, and cleared
    for (int q = tid; q < half + nw; q += nthr) {
      uint32_t acc = lds[q];
      for (int w = 1; w < waves; ++w) {
        uint32_t *src = lds + size_t(w) * words + q;
        acc = q < half ? acc + *src : acc | *src;
        *src = 0u;
      }
      lds[q] = acc;
    }
    __syncthreads();
    if (tid < kWave)
      emit_row(lds, lds + half, reinterpret_cast<uint16_t *>(lds + half + nw), nw, K, d.d_ent + d.d_cap[dd] + 1u,
               e - b, lane);
  }
  __syncthreads();  // every table is clear again
}

// D rebuild (Sec. 4.3): per document gather the new topics through the
// inverted index (doc order -> word-order slot) into a per-wave LDS table of
// 16-bit counts, marking each touched topic in a bitmap.  The row is then
// emitted in ascending topic order: each lane expands one bitmap word into a
// list of topics at its prefix-sum offset, and one lane per listed topic
// writes the packed entry.  The work per document is K/2048 wave steps plus
// about one per 32 touched topics, so it follows the tokens, not K.
__global__ __launch_bounds__(kBlock) void k_rebuild_d(DevState d, Params p, int light) {
  extern __shared__ uint32_t ldsu[];
  const int K = p.K;
  const int half = (K + 1) / 2, nw = (K + 31) / 32;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  uint32_t *hist = ldsu + size_t(wave) * d_rebuild_lds_words(K);
  uint32_t *bits = hist + half;
  uint16_t *list = reinterpret_cast<uint16_t *>(bits + nw);
  for (int q = lane; q < half; q += kWave) hist[q] = 0u;
  for (int q = lane; q < nw; q += kWave) bits[q] = 0u;
  uint32_t bad = 0;
  // the heavy documents first, each by the whole workgroup (wave 0's tables shared)
  if (p.n_heavy)
    heavy_rebuild_d(d, p, ldsu, bad);
  int part = light ? 0 : kXcds;  // heavy only: the light documents are k_rebuild_d_sort's
  for (;;) {
    uint32_t d0 = 0, d1 = 0;
    if (!next_docs(d.counters + CNT_REBUILD_D, p, part, lane, d0, d1)) break;
    const int nb = int(d1 - d0);
    // the batch's document offsets and D-row offsets, one per lane (loaded
    // here so that no later wait for them also waits for the prefetches)
    const uint32_t b_all = lane <= nb ? d.doc_off[d0 + uint32_t(lane)] : 0u;
    const uint32_t cap_all = lane < nb ? d.d_cap[d0 + uint32_t(lane)] : 0u;
    const uint32_t e_all = uint32_t(__shfl_down(int(b_all), 1, kWave));
    // the batch's light documents moved to the first lanes (a heavy one is a
    // workgroup's, heavy_rebuild_d), so that the loop below has no branch
    // around them: lane j holds begin, end and D-row offset of light document j
    const bool light = lane < nb && e_all - b_all <= kHeavyDoc;
    const unsigned long long lm = __ballot(light);
    const int nd = __popcll(lm);
    const uint32_t below = __builtin_amdgcn_mbcnt_hi(uint32_t(lm >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(lm), 0u));
    const uint32_t target = light ? below : uint32_t(nd) + (uint32_t(lane) - below);  // distinct lanes
    const uint32_t bv = uint32_t(__builtin_amdgcn_ds_permute(int(target * 4u), int(b_all)));
    const uint32_t ev = uint32_t(__builtin_amdgcn_ds_permute(int(target * 4u), int(e_all)));
    const uint32_t capv = uint32_t(__builtin_amdgcn_ds_permute(int(target * 4u), int(cap_all)));
    // pipeline over the first kPre*64 tokens of each document: the
    // word-order slots of document i+3 and the topics of document i+2 are
    // loaded while document i is processed.  Every load is issued (slot
    // indexes past the batch are clamped; lanes past a document's end read
    // slot 0's topic), so the waits count a fixed number of loads and do not
    // drain the pipeline.
    const uint32_t last = uint32_t(p.n - 1);
    auto slots_of = [&](int doc, uint32_t (&w)[kPre]) {
      const uint32_t bn = __builtin_amdgcn_readlane(bv, doc);
#pragma unroll
      for (int c = 0; c < kPre; ++c) w[c] = d.dt_wpos[min(bn + uint32_t(c * kWave + lane), last)];
    };
    auto topics_of = [&](int doc, const uint32_t (&w)[kPre], uint32_t (&z)[kPre]) {
      const uint32_t bn = __builtin_amdgcn_readlane(bv, doc), en = __builtin_amdgcn_readlane(ev, doc);
#pragma unroll
      for (int c = 0; c < kPre; ++c) z[c] = d.z_w[bn + uint32_t(c * kWave + lane) < en ? w[c] : 0u];
    };
    uint32_t zA[kPre], zB[kPre], wC[kPre], wD[kPre];
    slots_of(0, wD);
    topics_of(0, wD, zA);
    slots_of(1, wD);
    topics_of(1, wD, zB);
    slots_of(2, wC);
    for (int i = 0; i < nd; ++i) {
      const uint32_t b = __builtin_amdgcn_readlane(bv, i), e = __builtin_amdgcn_readlane(ev, i);
      uint32_t zv[kPre];
#pragma unroll
      for (int c = 0; c < kPre; ++c) {
        zv[c] = zA[c];
        zA[c] = zB[c];
      }
      slots_of(i + 3, wD);
      topics_of(i + 2, wC, zB);
#pragma unroll
      for (int c = 0; c < kPre; ++c) wC[c] = wD[c];
#pragma unroll
      for (int c = 0; c < kPre; ++c) {
        if (b + uint32_t(c * kWave + lane) < e) {
          const uint32_t z = zv[c];
          if (z < uint32_t(K)) {
            atomicAdd(&hist[z >> 1], (z & 1u) ? 0x10000u : 1u);
            atomicOr(&bits[z >> 5], 1u << (z & 31u));
          } else {
            bad++;
          }
        }
      }
      // the rest of a long document, kTail chunks at a time: all their slot
      // loads, then all their topic gathers, are in flight together
      for (uint32_t p0 = b + uint32_t(kPre * kWave); p0 < e; p0 += uint32_t(kTail * kWave)) {
        uint32_t zt[kTail];
#pragma unroll
        for (int c = 0; c < kTail; ++c) {
          const uint32_t pp = p0 + uint32_t(c * kWave + lane);
          zt[c] = pp < e ? d.dt_wpos[pp] : 0u;
        }
#pragma unroll
        for (int c = 0; c < kTail; ++c) {
          const uint32_t pp = p0 + uint32_t(c * kWave + lane);
          if (pp < e) zt[c] = d.z_w[zt[c]];
        }
#pragma unroll
        for (int c = 0; c < kTail; ++c) {
          if (p0 + uint32_t(c * kWave + lane) < e) {
            const uint32_t z = zt[c];
            if (z < uint32_t(K)) {
              atomicAdd(&hist[z >> 1], (z & 1u) ? 0x10000u : 1u);
              atomicOr(&bits[z >> 5], 1u << (z & 31u));
            } else {
              bad++;
            }
          }
        }
      }
      __threadfence_block();
      // (readlane returns a signed int: the offset is taken back to unsigned,
      // since D has more than 2^31 slots on the largest corpora)
      emit_row(hist, bits, list, nw, K, d.d_ent + uint32_t(__builtin_amdgcn_readlane(capv, i)) + 1u, e - b, lane);
    }
  }
  if (bad) atomicAdd(&d.stats[ST_ERRORS], (unsigned long long)bad);
}

// The D rows of the light documents for large K, one wave per document
// without a table of K counts (which leaves room for two waves per CU at
// K = 32,768): the wave gathers the document's topics into its LDS buffer,
// sorts them (bitonic, ascending; topics >= K are errors and sort last as
// 0xFFFF), and writes one entry per run of equal topics.  The rows are the
// ones emit_row writes: entries in ascending topic order, padding entries
// of topic K, the header (length << 16 | entries).
constexpr int kSortGather = 8;  // slots per lane whose loads are in flight together

// Bitonic sort (ascending) of the P = 64 * E slots of sz in registers: lane l
// holds slots l * E .. l * E + E - 1; compare-exchanges between slots of one
// lane stay in registers, those between lanes exchange by shuffle.  The same
// network as the sort in LDS below, so the same result.
template <int E>
__device__ __forceinline__ void sort_in_registers(uint16_t *__restrict__ sz, int lane) {
  constexpr uint32_t P = uint32_t(E) * uint32_t(kWave);
  uint32_t x[E];
#pragma unroll
  for (int r = 0; r < E; ++r) x[r] = sz[lane * E + r];
#pragma unroll
  for (uint32_t size = 2; size <= P; size <<= 1) {
#pragma unroll
    for (uint32_t stride = size >> 1; stride > 0; stride >>= 1) {
      if (stride < uint32_t(E)) {
#pragma unroll
        for (int r = 0; r < E; ++r) {
          if ((uint32_t(r) & stride) == 0u) {
            const int q = r | int(stride);
            const bool asc = (uint32_t(lane * E + r) & size) == 0u;
            const uint32_t lo = min(x[r], x[q]), hi = max(x[r], x[q]);
            x[r] = asc ? lo : hi;
            x[q] = asc ? hi : lo;
          }
        }
      } else {
        const int dl = int(stride / uint32_t(E));        // partner lane distance
        const bool upper = (lane & dl) != 0;             // this lane holds the higher slot
        const bool asc = (uint32_t(lane * E) & size) == 0u;
#pragma unroll
        for (int r = 0; r < E; ++r) {
          const uint32_t o = uint32_t(__shfl_xor(int(x[r]), dl, kWave));
          x[r] = (asc != upper) ? min(x[r], o) : max(x[r], o);
        }
      }
    }
  }
#pragma unroll
  for (int r = 0; r < E; ++r) sz[lane * E + r] = uint16_t(x[r]);
}
__global__ __launch_bounds__(kBlock) void k_rebuild_d_sort(DevState d, Params p) {
  extern __shared__ uint32_t ldsu[];
  const int K = p.K;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  uint16_t *sz = reinterpret_cast<uint16_t *>(ldsu) + size_t(wave) * kHeavyDoc;
  uint32_t bad = 0;
  int part = 0;
  for (;;) {
    uint32_t d0 = 0, d1 = 0;
    if (!next_docs(d.counters + CNT_REBUILD_D, p, part, lane, d0, d1)) break;
    for (uint32_t dd = d0; dd < d1; ++dd) {
      const uint32_t b = d.doc_off[dd], len = d.doc_off[dd + 1] - b;
      if (len > uint32_t(kHeavyDoc)) continue;  // a heavy document: k_rebuild_d's
      uint32_t P = kWave;
      while (P < len) P <<= 1;
      // the topics, kSortGather slots per lane at a time (slot loads, then gathers)
      for (uint32_t q0 = 0; q0 < P; q0 += uint32_t(kSortGather * kWave)) {
        uint32_t zz[kSortGather];
#pragma unroll
        for (int c = 0; c < kSortGather; ++c) {
          const uint32_t q = q0 + uint32_t(c * kWave + lane);
          zz[c] = q < len ? d.dt_wpos[b + q] : 0u;
        }
#pragma unroll
        for (int c = 0; c < kSortGather; ++c) {
          const uint32_t q = q0 + uint32_t(c * kWave + lane);
          if (q < len) zz[c] = d.z_w[zz[c]];
        }
#pragma unroll
        for (int c = 0; c < kSortGather; ++c) {
          const uint32_t q = q0 + uint32_t(c * kWave + lane);
          if (q < P) {
            uint32_t z = 0xFFFFu;
            if (q < len) {
              if (zz[c] < uint32_t(K)) z = zz[c];
              else bad++;
            }
            sz[q] = uint16_t(z);
          }
        }
      }
      __threadfence_block();
      // bitonic sort of the P slots, ascending: in registers up to 512 slots
      if (P <= 512u) {
        if (P == 64u) sort_in_registers<1>(sz, lane);
        else if (P == 128u) sort_in_registers<2>(sz, lane);
        else if (P == 256u) sort_in_registers<4>(sz, lane);
        else sort_in_registers<8>(sz, lane);
        __threadfence_block();
      }
      for (uint32_t size = 2; P > 512u && size <= P; size <<= 1) {
        for (uint32_t stride = size >> 1; stride > 0; stride >>= 1) {
          for (uint32_t t = uint32_t(lane); t < P / 2; t += kWave) {
            const uint32_t i = 2 * t - (t & (stride - 1)), j = i + stride;
            const uint32_t a = sz[i], c = sz[j];
            if ((a > c) == ((i & size) == 0)) {
              sz[i] = uint16_t(c);
              sz[j] = uint16_t(a);
            }
          }
          __threadfence_block();
        }
      }
      // entries: a run starts where the topic changes; first the number of
      // entries, then the runs from the last 64 slots to the first, so that
      // each run's end (the next run's start) is known
      uint32_t nnz = 0;
      for (uint32_t q0 = 0; q0 < len; q0 += kWave) {
        const uint32_t i = q0 + uint32_t(lane);
        const uint32_t zi = i < len ? sz[i] : 0xFFFFu, zp = i > 0 && i < len ? sz[i - 1] : 0xFFFFFFFFu;
        nnz += uint32_t(__popcll(__ballot(i < len && zi != 0xFFFFu && zi != zp)));
      }
      uint32_t *out = d.d_ent + d.d_cap[dd] + 1u;
      uint32_t after = nnz, next = len;  // entries and first run start past the current 64 slots
      for (int q0 = int((len - 1u) & ~uint32_t(kWave - 1)); q0 >= 0; q0 -= kWave) {
        const uint32_t i = uint32_t(q0 + lane);
        const uint32_t zi = i < len ? sz[i] : 0xFFFFu, zp = i > 0 && i < len ? sz[i - 1] : 0xFFFFFFFFu;
        const bool start = i < len && zi != zp;
        const unsigned long long sm = __ballot(start), em = __ballot(start && zi != 0xFFFFu);
        const unsigned long long above = lane == kWave - 1 ? 0ull : sm & (~0ull << (lane + 1));
        const uint32_t end = above ? uint32_t(q0) + uint32_t(__ffsll(above) - 1) : next;
        const uint32_t n_here = uint32_t(__popcll(em));
        if (start && zi != 0xFFFFu) {
          const uint32_t below = uint32_t(__popcll(em & ((1ull << lane) - 1ull)));
          out[after - n_here + below] = (zi << 16) | (end - i);
        }
        after -= n_here;
        next = sm ? uint32_t(q0) + uint32_t(__ffsll(sm) - 1) : next;
      }
      for (uint32_t q = nnz + uint32_t(lane); q + 1u < d_row_slots(nnz); q += kWave) out[q] = uint32_t(K) << 16;
      if (lane == 0) out[-1] = (len << 16) | nnz;
      __threadfence_block();
    }
  }
  if (bad) atomicAdd(&d.stats[ST_ERRORS], (unsigned long long)bad);
}

// LLPT terms (Sec. 2.2): for every token,
//   log2( (sum_{k in nz(D[d])} D[d][k] W^[v][k] + alpha * sum_k W^[v][k]) / (len(d) + K alpha) ),
// summed per unit of the sampler (per batch of light regions) in an order that
// the layout fixes, so that the result does not depend on the schedule.
//
// The work is the sampler's S' pass without the draws, and it is organised the
// same way: batches of 64 tokens per wave, rows in registers by groups of 4, 8
// or 16 lanes, then one lane per token for the logarithm.  A 16-lane loop per
// token, 4 waves per CU from K = 10,000 on and the rows in global memory at
// K = 32,768 took 18.6 ms for 144M tokens at K = 1,000, 25.6 ms for 33M at
// 10,000 and 74.3 ms for 20M at 32,768; these take 5.9, 6.7 and 10.5 ms.
__device__ __forceinline__ double llpt_term(double s, double asw, uint32_t len, double Kalpha) {
  return log2((s + asw) / (double(len) + Kalpha));
}

template <int NB>
__device__ __forceinline__ void loglik_body(DevState d, Params p) {
  extern __shared__ double lds[];
  const int K = p.K;
  double *wh = lds;                     // [wh_entries(K)]: W^ of the region's word, zeros past K
  double *s_u = lds + wh_entries(K);    // [NB]
  double *s_part = s_u + NB;            // [NB / kWave]
  uint32_t *s_off = reinterpret_cast<uint32_t *>(s_part + NB / kWave);
  uint32_t *s_nnz = s_off + NB;
  uint32_t *s_reg = s_nnz + NB;         // [4]: the region's index (or past the end), word, begin, end
  uint8_t *s_list = reinterpret_cast<uint8_t *>(s_reg + 4);
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const BatchLds bt{s_off + wave * kWave, s_nnz + wave * kWave, s_u + wave * kWave, nullptr, nullptr,
                    s_list + wave * kWave};
  const double Kalpha = double(K) * p.alpha;
  for (int k = K + tid; k < wh_entries(K); k += NB) wh[k] = 0.0;
  uint32_t cur = 0xFFFFFFFFu;
  double asw = 0.0;
  const uint32_t *held = nullptr;  // as in the sampler: the sparse word whose row wh holds
  uint32_t held_nnz = 0;
  for (;;) {
    if (tid == 0) {
      const uint32_t r = atomicAdd(&d.counters[CNT_LOGLIK], 1u);
      s_reg[0] = r;
      if (int64_t(r) < p.n_units) {
        s_reg[1] = d.unit[3 * size_t(r)] & ~kUnitContinues;
        s_reg[2] = d.unit[3 * size_t(r) + 1];
        s_reg[3] = d.unit[3 * size_t(r) + 2];
      }
    }
    __syncthreads();
    const uint32_t r = __builtin_amdgcn_readfirstlane(s_reg[0]);
    if (int64_t(r) >= p.n_units) break;
    const uint32_t v = __builtin_amdgcn_readfirstlane(s_reg[1]);
    const uint32_t b = __builtin_amdgcn_readfirstlane(s_reg[2]), e = __builtin_amdgcn_readfirstlane(s_reg[3]);
    if (v != cur) {
      cur = v;
      asw = p.alpha * d.wrec[v].sumw;
      if (int32_t(v) < p.n_dense) {
        const int32_t *wrow = d.w_dense + size_t(v) * size_t(K);
        for (int k = tid; k < K; k += NB) wh[k] = what(uint32_t(wrow[k]), p.beta, d.den[k]);
        held = nullptr;
      } else {
        const int s = int(v) - p.n_dense;
        const uint32_t *ents = d.ws_ent + d.ws_cap[s];
        const uint32_t nnz = d.ws_nnz[s];
        if (held) {
          for (uint32_t q = tid; q < held_nnz; q += NB) {
            const uint32_t k = held[q] >> 16;
            wh[k] = d.bden[k];
          }
        } else {
          for (int k = tid; k < K; k += NB) wh[k] = d.bden[k];
        }
        __syncthreads();
        for (uint32_t q = tid; q < nnz; q += NB) {
          const uint32_t ent = ents[q];
          wh[ent >> 16] = what(ent & 0xFFFFu, p.beta, d.den[ent >> 16]);
        }
        held = ents;
        held_nnz = nnz;
      }
      __syncthreads();
    }
    const WordState w{wh, nullptr, 0, K, 0, 0u, 0.0, 0.0, p.alpha, nullptr, nullptr};
    const uint32_t bsz = min(uint32_t(kWave), max(16u, ((e - b + uint32_t(NB / kWave) - 1u) / uint32_t(NB / kWave) + 15u) & ~15u));
    double part = 0.0;  // this lane's tokens of the region
    for (uint32_t base = b + uint32_t(wave) * bsz; base < e; base += uint32_t(NB / kWave) * bsz) {
      const int ln = lane_here();
      const uint32_t j = base + uint32_t(ln);
      const bool in = j < min(e, base + bsz);
      uint32_t off = 0, hdr = 0;
      if (in) {
        off = d.wt_kr[j].y;
        hdr = d.d_ent[off];
        bt.off[ln] = off;
        bt.nnz[ln] = hdr & 0xFFFFu;
      }
      uint32_t none = 0;
      uint32_t nnz_read;
      draw_tokens<(NB >= 1024), true>(in, off, hdr & 0xFFFFu, 0, ln, bt, w, d.d_ent, none, &nnz_read);
      if (in) part += llpt_term(bt.u[ln], asw, hdr >> 16, Kalpha);
    }
    part = group_sum<kWave>(part);
    if (lane == 0) s_part[wave] = part;
    __syncthreads();
    if (tid == 0) {
      double s = 0.0;
      for (int q = 0; q < NB / kWave; ++q) s += s_part[q];
      d.ll_part[r] = s;
    }
    // s_reg and s_part are next written behind the barrier that follows the fetch, by then read
    __syncthreads();
  }
}
__global__ __launch_bounds__(256, 7) void k_loglik(DevState d, Params p) { loglik_body<256>(d, p); }
__global__ __launch_bounds__(512, 4) void k_loglik_512(DevState d, Params p) { loglik_body<512>(d, p); }
__global__ __launch_bounds__(1024, 4) void k_loglik_1024(DevState d, Params p) { loglik_body<1024>(d, p); }

// The light regions, in the light sampler's batches, one wave each: partial
// p.n_units + i is batch i's.
__global__ __launch_bounds__(64, 4) void k_loglik_light(DevState d, Params p) {
  extern __shared__ double lds[];
  const int K = p.K;
  double *wh = lds;
  double *s_u = lds + wh_entries(K);
  uint32_t *s_off = reinterpret_cast<uint32_t *>(s_u + kWave);
  uint32_t *s_nnz = s_off + kWave;
  uint8_t *s_list = reinterpret_cast<uint8_t *>(s_nnz + kWave);
  const BatchLds bt{s_off, s_nnz, s_u, nullptr, nullptr, s_list};
  const int lane = threadIdx.x;
  const double Kalpha = double(K) * p.alpha;
  for (int k = K + lane; k < wh_entries(K); k += kWave) wh[k] = 0.0;
  int held = -1;  // as in k_sampler_light
  uint32_t held_k = 0;
  double held_b = 0.0;
  auto order = [&]() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); };
  for (uint32_t bi = blockIdx.x; bi < uint32_t(p.n_light_batches); bi += gridDim.x) {
    const uint32_t r0 = __builtin_amdgcn_readfirstlane(d.light_batch[bi]);
    const int nw = int(__builtin_amdgcn_readfirstlane(d.light_batch[bi + 1]) - r0);  // 1..64
    const size_t rr = 3 * (size_t(p.light_begin) + r0 + uint32_t(min(lane, nw - 1)));
    const uint32_t v_l = d.region[rr], b_l = d.region[rr + 1], e_l = d.region[rr + 2];
    const uint32_t b0 = __builtin_amdgcn_readlane(b_l, 0), e0 = __builtin_amdgcn_readlane(e_l, nw - 1);
    const int ln = lane_here();
    const uint32_t j = b0 + uint32_t(ln);
    const bool in = j < e0;
    uint32_t off = 0, hdr = 0;
    if (in) off = d.wt_kr[j].y;
    const bool dense_l = int32_t(v_l) < p.n_dense;
    const int s_l = dense_l ? 0 : int(v_l) - p.n_dense;
    const uint32_t nnz_l = dense_l ? 0u : d.ws_nnz[s_l];
    const uint32_t cap_l = dense_l ? 0u : d.ws_cap[s_l];
    if (in) {
      hdr = d.d_ent[off];
      bt.off[ln] = off;
      bt.nnz[ln] = hdr & 0xFFFFu;
    }
    auto entry_of = [&](int i) {
      const uint32_t n = __builtin_amdgcn_readlane(nnz_l, i), c = __builtin_amdgcn_readlane(cap_l, i);
      return uint32_t(lane) < n ? d.ws_ent[c + uint32_t(lane)] : 0u;
    };
    const double sumw_l = d.wrec[v_l].sumw;
    uint32_t ent_1 = entry_of(0), ent_2 = entry_of(min(1, nw - 1));
    double den_1 = d.den[ent_1 >> 16], bden_1 = d.bden[ent_1 >> 16];
    double part = 0.0;
    for (int i = 0; i < nw; ++i) {
      const uint32_t v = __builtin_amdgcn_readlane(v_l, i);
      const uint32_t ent = ent_1;
      const double den_e = den_1, bden_e = bden_1;
      ent_1 = ent_2;
      den_1 = d.den[ent_1 >> 16];
      bden_1 = d.bden[ent_1 >> 16];
      ent_2 = entry_of(min(i + 2, nw - 1));
      const int f = int(__builtin_amdgcn_readlane(b_l, i) - b0), l = int(__builtin_amdgcn_readlane(e_l, i) - b0);
      const bool mine = ln >= f && ln < l;
      const double asw = p.alpha * readlane_f64(sumw_l, i);
      if (int32_t(v) < p.n_dense) {
        const int32_t *wrow = d.w_dense + size_t(v) * size_t(K);
        fill_dense_wave(wrow, d.den, p.beta, K, lane, wh);
        held = -1;
      } else {
        const uint32_t n = __builtin_amdgcn_readlane(nnz_l, i);
        const uint32_t ek = ent >> 16;
        const double we = uint32_t(lane) < n ? what(ent & 0xFFFFu, p.beta, den_e) : 0.0;
        if (held >= 0) {
          if (lane < held) wh[held_k] = held_b;
        } else {
          for (int k = lane; k < K; k += kWave) wh[k] = d.bden[k];
        }
        order();
        if (uint32_t(lane) < n) wh[ek] = we;
        held = int(n);
        held_k = ek;
        held_b = bden_e;
      }
      order();
      const WordState w{wh, nullptr, 0, K, 0, 0u, 0.0, 0.0, p.alpha, nullptr, nullptr};
      uint32_t none = 0;
      uint32_t nnz_read;
      draw_tokens<false, true>(mine, off, hdr & 0xFFFFu, f, ln, bt, w, d.d_ent, none, &nnz_read);
      if (mine) part = llpt_term(bt.u[ln], asw, hdr >> 16, Kalpha);
      order();
    }
    part = group_sum<kWave>(part);
    if (lane == 0) d.ll_part[p.n_units + int64_t(bi)] = part;
  }
}

// Large K: the row in two tiles.  Pass 0 keeps each token's sum over the topics
// below KT and the chunk where its row reaches KT (in the workgroup's slice of
// ts_s and ts_code), pass 1 adds the topics from KT on, reading the row from
// that chunk.
__global__ __launch_bounds__(kTiledBlock) void k_loglik_tiled(DevState d, Params p) {
  extern __shared__ double lds[];
  const int K = p.K;
  const uint32_t kt = uint32_t(p.tile_topics);
  double *wt = lds;                                                    // [kt + kGroup]
  double *s_part = lds + kt + kGroup;                                  // [waves]
  uint32_t *s_reg = reinterpret_cast<uint32_t *>(s_part + kTiledBlock / kWave);  // [4]
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wave = tid / kWave, grp = lane / kGroup, li = lane % kGroup;
  const uint32_t pad = uint32_t(K) << 16;
  double *sc_s = d.ts_s + size_t(blockIdx.x) * size_t(p.max_region);
  uint32_t *sc_c = d.ts_code + size_t(blockIdx.x) * size_t(p.max_region);
  const double Kalpha = double(K) * p.alpha;
  const int waves = kTiledBlock / kWave;
  for (;;) {
    if (tid == 0) {
      const uint32_t r = atomicAdd(&d.counters[CNT_LOGLIK], 1u);
      s_reg[0] = r;
      if (int64_t(r) < p.n_regions) {
        s_reg[1] = d.region[3 * size_t(r)];
        s_reg[2] = d.region[3 * size_t(r) + 1];
        s_reg[3] = d.region[3 * size_t(r) + 2];
      }
    }
    __syncthreads();
    const uint32_t r = __builtin_amdgcn_readfirstlane(s_reg[0]);
    if (int64_t(r) >= p.n_regions) break;
    const uint32_t v = __builtin_amdgcn_readfirstlane(s_reg[1]);
    const uint32_t b = __builtin_amdgcn_readfirstlane(s_reg[2]), e = __builtin_amdgcn_readfirstlane(s_reg[3]);
    const double asw = p.alpha * d.wrec[v].sumw;
    double part = 0.0;
    for (int pass = 0; pass < 2; ++pass) {
      const uint32_t tbase = pass == 1 ? kt : 0u;
      const uint32_t tlen = pass == 1 ? uint32_t(K) + 1u - kt : kt;
      fill_tile(d, p, v, 0xFFFFFFFFu, tbase, tlen, kt, wt, tid, kTiledBlock);  // no topic left out
      const TileState ts{wt, tbase, kt, 0u - tbase * 8u};
      const uint32_t stride = uint32_t(waves) * 4u;
      uint32_t off_n = d.wt_kr[min(b + uint32_t(wave) * 4u + uint32_t(grp), e - 1u)].y;
      for (uint32_t j0 = b + uint32_t(wave) * 4u; j0 < e; j0 += stride) {
        const uint32_t j = j0 + uint32_t(grp), q = j - b;
        const uint32_t off = off_n;
        if (j0 + stride < e) off_n = d.wt_kr[min(j + stride, e - 1u)].y;  // one step ahead
        if (j >= e) continue;
        const uint32_t *row = d.d_ent + off;
        const uint32_t hdr = row[0], slots = d_row_slots(hdr & 0xFFFFu), nch = (slots + kChunk - 1) / kChunk;
        double s = 0.0;
        const uint32_t c_from = pass == 0 ? 0u : sc_c[q];
        uint32_t sc = c_from;
        bool open = true;
        for (uint32_t c0 = c_from; open; c0 += kTiledAhead) {
          uint32_t rr[kTiledAhead][kMaxRun];
#pragma unroll
          for (int c = 0; c < kTiledAhead; ++c) load_run_masked(row, c0 + uint32_t(c), slots, li, pad, rr[c]);
#pragma unroll
          for (int c = 0; c < kTiledAhead; ++c) {
            if (open) {
              sc = c0 + uint32_t(c);
              open = sc + 1u < nch;
              if (pass == 0) open = open && (uint32_t(__shfl(int(rr[c][kMaxRun - 1]), kGroup - 1, kGroup)) >> 16) < kt;
              s += run_sum_tile(rr[c], ts);
            }
          }
        }
        s = gsum<kGroup>(s);
        if (li == 0) {
          if (pass == 0) {
            sc_s[q] = s;
            sc_c[q] = sc;
          } else {
            part += llpt_term(sc_s[q] + s, asw, hdr >> 16, Kalpha);
          }
        }
      }
      __syncthreads();
    }
    part = group_sum<kWave>(part);
    if (lane == 0) s_part[wave] = part;
    __syncthreads();
    if (tid == 0) {
      double s = 0.0;
      for (int q = 0; q < waves; ++q) s += s_part[q];
      d.ll_part[r] = s;
    }
    __syncthreads();
  }
}

// out[0] = sum of part[0..n), one workgroup in a fixed order: 256 strands of
// every 256th value each, kSumAhead of them loaded together.
constexpr int kSumAhead = 16;
__global__ __launch_bounds__(kBlock) void k_loglik_reduce(const double *__restrict__ part, int64_t n,
                                                          double *__restrict__ out) {
  __shared__ double red[kBlock / kWave];
  double s = 0.0;
  int64_t q = threadIdx.x;
  for (; q + int64_t(kSumAhead - 1) * kBlock < n; q += int64_t(kSumAhead) * kBlock) {
    double v[kSumAhead];
#pragma unroll
    for (int u = 0; u < kSumAhead; ++u) v[u] = part[q + int64_t(u) * kBlock];
#pragma unroll
    for (int u = 0; u < kSumAhead; ++u) s += v[u];
  }
  for (; q < n; q += kBlock) s += part[q];
  s = block_sum(s, red);
  if (threadIdx.x == 0) out[0] = s;
}

}  // namespace

// ---------------------------------------------------------- launchers ----

// Dynamic LDS above 64 KB per workgroup has to be requested for the kernel.
template <typename F>
hipError_t allow_lds(F *kernel, size_t bytes) {
  if (bytes <= 65536) return hipSuccess;
  return hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                             int(bytes));
}

hipError_t launch_init_topics(const DevState &d, const Params &p, hipStream_t s) {
  const int64_t blocks = std::min<int64_t>((p.n + kBlock - 1) / kBlock, int64_t(p.grid_docs) * 8);
  hipLaunchKernelGGL(k_init_topics, dim3(uint32_t(blocks)), dim3(kBlock), 0, s, d.wt_kr, d.z_w, p.n, p.K, p.seed);
  return hipGetLastError();
}

hipError_t launch_clear_skips(const DevState &d, const Params &p, uint32_t t, hipStream_t s, bool reset_count) {
  const int64_t n = skip_words(p.n);
  const int64_t blocks = std::min<int64_t>((n + kBlock - 1) / kBlock, int64_t(p.grid_docs) * 4);
  hipLaunchKernelGGL(k_clear_skips, dim3(uint32_t(std::max<int64_t>(blocks, 1))), dim3(kBlock), 0, s, d.skip_bits,
                     d.skip_doc, n, n + 64, d.skip_hist, t, reset_count ? 1 : 0);
  return hipGetLastError();
}

hipError_t launch_reset_counters(uint32_t *counters, hipStream_t s) {
  hipLaunchKernelGGL(k_reset_counters, dim3(1), dim3(kBlock), 0, s, counters);
  return hipGetLastError();
}

hipError_t launch_begin_iteration(const DevState &d, const Params &p, hipStream_t s) {
  hipLaunchKernelGGL(k_begin, dim3((p.K + kBlock - 1) / kBlock), dim3(kBlock), 0, s, d.T, d.den, d.bden, p.K, p.beta,
                     p.vbeta, d.counters, d.stats);
  return hipGetLastError();
}

hipError_t launch_beta_sum(const DevState &d, const Params &p, hipStream_t s) {
  hipLaunchKernelGGL(k_beta_sum, dim3(1), dim3(kBlock), 0, s, d, p);
  return hipGetLastError();
}
hipError_t launch_word_pre(const DevState &d, const Params &p, hipStream_t s) {
  if (p.f32) {
    const auto base = q_block_topics(p.sampler_block) == 16 ? k_block_base<16> : k_block_base<32>;
    hipLaunchKernelGGL(base, dim3(uint32_t((p.K + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, d, p);
    const hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
  }
  if (p.sparse_pre) {
    // the topic list and the sum of beta/den[k] follow the current T
    hipError_t err;
    if (p.K < kWBitsK) {
      const uint32_t grid = uint32_t((p.K + kListTopics - 1) / kListTopics) + 1u;
      hipLaunchKernelGGL(k_topic_list, dim3(grid), dim3(kBlock), sizeof(uint32_t) * size_t((p.K + 3) & ~3), s, d, p);
      err = hipGetLastError();
    } else {
      size_t bytes = d.topic_tmp_bytes;
      err = sort_pairs_u32(d.topic_tmp, bytes, d.T, d.topic_keys, d.topic_iota, d.topic_order, p.K, 32, s);
      if (err == hipSuccess) err = launch_beta_sum(d, p, s);
    }
    if (err != hipSuccess) return err;
    if (p.small_begin < p.n_present) {
      const int per = kBlock / kGroup;
      hipLaunchKernelGGL(k_word_pre_small, dim3(uint32_t((p.n_present - p.small_begin + per - 1) / per)), dim3(kBlock),
                         0, s, d, p);
      if ((err = hipGetLastError()) != hipSuccess) return err;
    }
  }
  // without the topic list a table of K 16-bit counts per wave (K below
  // 4,096: at most 32 KB), for sparse rows only
  const size_t lds = p.sparse_pre || p.n_dense >= p.n_present ? 0 : sizeof(uint16_t) * size_t((p.K + 1) & ~1) * (kBlock / kWave);
  const int32_t words = p.sparse_pre ? p.small_begin : p.n_present;
  if (words == 0) return hipSuccess;
  const uint32_t grid = uint32_t((words + kBlock / kWave - 1) / (kBlock / kWave));
  hipLaunchKernelGGL(k_word_pre_wave, dim3(grid), dim3(kBlock), lds, s, d, p);
  return hipGetLastError();
}

hipError_t launch_doc_pass(const DevState &d, const Params &p, uint32_t t, hipStream_t s) {
  const size_t lds = sizeof(uint16_t) * size_t(p.K) * size_t(p.doc_waves);
  const auto kernel = p.key_identity ? k_doc_pass<true> : k_doc_pass<false>;
  hipError_t err = allow_lds(kernel, lds);
  if (err != hipSuccess) return err;
  hipLaunchKernelGGL(kernel, dim3(doc_pass_grid(p)), dim3(kWave * p.doc_waves), lds, s, d, p, t, d.stats);
  return hipGetLastError();
}

// The sampler's dynamic LDS for K topics and workgroups of nb threads: the
// W^' row, the Q' block prefix, the per-wave batch slices (u, row offset,
// length, drawn topic, list place; the long-row hand-off) and the region.
size_t sampler_lds_bytes(int K, int nb, bool q_table) {
  const size_t blocks = size_t((K + kGroup - 1) / kGroup);
  const size_t words = size_t(wh_entries(K)) + size_t(q_blocks_padded(int(blocks))) + 1;
  size_t bytes = sizeof(double) * words + size_t(nb) * (sizeof(double) + 2 * sizeof(uint32_t) + sizeof(uint16_t) + 1) +
                 sizeof(uint32_t) * (size_t(nb) / kGroup * kMaxRun + 4);
  if (q_table) bytes += blocks * (kQwStride * sizeof(double) + 1);
  return bytes;
}

// Resident waves per CU of a kernel with workgroups of nb threads and this
// dynamic LDS (0 if it does not fit).
template <typename F>
static int resident_waves(F *kernel, int nb, size_t lds) {
  int blocks = 0;
  hipError_t err = allow_lds(kernel, lds);
  if (err == hipSuccess) err = hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, kernel, nb, lds);
  (void)hipGetLastError();
  return err == hipSuccess ? blocks * nb / kWave : 0;
}
// Whether the fp64 sampler (256 threads) keeps the per-topic partial sums of
// the Q' blocks in LDS (q_draw's search instead of its walk; the same draws):
// when they leave it as many resident waves.
bool sampler_q_table(int K) {
  return resident_waves(k_sampler, kBlock, sampler_lds_bytes(K, kBlock, true)) >=
         resident_waves(k_sampler, kBlock, sampler_lds_bytes(K, kBlock, false));
}

// The single-precision sampler's dynamic LDS, and its workgroup size for K
// topics: `want` when nonzero, else the size with the most resident waves per
// CU (ties to the smaller).
size_t sampler_f_lds_bytes(int K, int nb) {
  const size_t blocks = size_t((K + q_block_topics(nb) - 1) / q_block_topics(nb));
  return sizeof(float) * size_t(wf_entries(K)) + sizeof(double) * (blocks + 1) +
         size_t(nb) * (sizeof(double) + 2 * sizeof(uint32_t) + sizeof(uint16_t) + 1) + 4 * sizeof(uint32_t);
}
int sampler_f_block(int K, int want) {
  int best = 0, best_waves = 0;
  for (const int nb : {256, 512, 1024}) {
    if (want && nb != want) continue;
    const int waves = resident_waves(nb == 1024 ? k_sampler_f_1024 : nb == 512 ? k_sampler_f_512 : k_sampler_f, nb,
                                     sampler_f_lds_bytes(K, nb));
    if (waves > best_waves) {
      best = nb;
      best_waves = waves;
    }
  }
  return best;
}

// hipSuccess if the kernel has no static LDS (its dynamic LDS starts at address 0).
static hipError_t no_static_lds(const void *kernel) {
  hipFuncAttributes a;
  const hipError_t e = hipFuncGetAttributes(&a, kernel);
  return e != hipSuccess ? e : a.sharedSizeBytes == 0 ? hipSuccess : hipErrorInvalidConfiguration;
}

int tiled_topics(int K) { return ((K + 2) / 2 + kGroup - 1) / kGroup * kGroup; }
hipError_t launch_sampler(const DevState &d, const Params &p, uint32_t t, hipStream_t s) {
  if (p.n_units == 0) return hipSuccess;  // every region is light
  const size_t lds = p.f32 ? sampler_f_lds_bytes(p.K, p.sampler_block) : sampler_lds_bytes(p.K, p.sampler_block, p.q_table != 0);
  const auto kernel = !p.f32 ? k_sampler
                      : p.sampler_block == 1024 ? k_sampler_f_1024
                      : p.sampler_block == 512  ? k_sampler_f_512
                                                : k_sampler_f;
  const hipError_t err = allow_lds(kernel, lds);
  if (err != hipSuccess) return err;
  hipLaunchKernelGGL(kernel, dim3(uint32_t(sampler_grid(p))), dim3(uint32_t(p.sampler_block)), lds, s, d, p, t, d.stats);
  return hipGetLastError();
}

// The light sampler's dynamic LDS for K topics (one wave).
size_t light_lds_bytes(int K) {
  const size_t nbp = size_t(q_blocks_padded((K + kGroup - 1) / kGroup));
  return sizeof(double) * (size_t(wh_entries(K)) + nbp + 1 + kWave) +
         size_t(kWave) * (2 * sizeof(uint32_t) + sizeof(uint16_t) + 1) + sizeof(uint32_t) * (kWave / kGroup * kMaxRun);
}

hipError_t launch_sampler_light(const DevState &d, const Params &p, uint32_t t, hipStream_t s) {
  if (p.n_light_batches <= 0) return hipSuccess;
  const size_t lds = light_lds_bytes(p.K);
  hipError_t err = allow_lds(k_sampler_light, lds);
  if (err != hipSuccess) return err;
  const uint32_t grid = uint32_t(light_grid(p));
  hipLaunchKernelGGL(k_sampler_light, dim3(grid), dim3(kWave), lds, s, d, p, t, d.stats);
  return hipGetLastError();
}

hipError_t launch_rebuild(const DevState &d, const Params &p, hipStream_t s, const StatSlots *slots) {
  hipError_t err = launch_zero_split(d, p, s, slots);
  if (err == hipSuccess) err = launch_rebuild_w(d, p, s);
  if (err == hipSuccess) err = launch_rebuild_d(d, p, s);
  return err;
}

hipError_t launch_zero_split(const DevState &d, const Params &p, hipStream_t s, const StatSlots *slots) {
  const int64_t zb = std::min<int64_t>((int64_t(p.n_dense) * p.K + kBlock - 1) / kBlock + kFoldBlocks, 65536);
  hipLaunchKernelGGL(k_zero_split, dim3(uint32_t(zb)), dim3(kBlock), 0, s, d, p, slots ? *slots : StatSlots{},
                     slots ? 1 : 0);
  return hipGetLastError();
}

hipError_t launch_fold_stats(const DevState &d, const StatSlots &slots, hipStream_t s) {
  hipLaunchKernelGGL(k_fold_stats, dim3(kFoldBlocks), dim3(kBlock), 0, s, d, slots);
  return hipGetLastError();
}

hipError_t launch_rebuild_w(const DevState &d, const Params &p, hipStream_t s) {
  hipError_t err;
  // large K: the bitmap variants, whose work follows the tokens instead of K
  const size_t nwords = size_t((p.K + 31) / 32);
  if (w_bits(p)) {
    // two 16-bit counts per word when every region is shorter than 2^16 tokens
    const bool packed = p.max_region > 0 && p.max_region < 65536;
    const size_t wlds = sizeof(uint32_t) * ((packed ? size_t(p.K + 1) / 2 : size_t(p.K)) + nwords);
    if (packed) {
      err = allow_lds(k_rebuild_w_bits<true>, wlds);
      if (err != hipSuccess) return err;
      hipLaunchKernelGGL(k_rebuild_w_bits<true>, dim3(uint32_t(p.grid_regions)), dim3(kBlock), wlds, s, d, p);
    } else {
      err = allow_lds(k_rebuild_w_bits<false>, wlds);
      if (err != hipSuccess) return err;
      hipLaunchKernelGGL(k_rebuild_w_bits<false>, dim3(uint32_t(p.grid_regions)), dim3(kBlock), wlds, s, d, p);
    }
    if ((err = hipGetLastError()) != hipSuccess) return err;
    // T: per-workgroup histograms
    if (!d.hist_rows) return hipErrorInvalidValue;  // allocated before any rebuild
    const int G = topic_hist_grid(p);
    uint32_t *rows = d.hist_rows;
    err = allow_lds(k_topic_hist, sizeof(uint32_t) * size_t(p.K));
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(k_topic_hist, dim3(uint32_t(G)), dim3(kHistBlock), sizeof(uint32_t) * size_t(p.K), s, d, p,
                       rows);
    if ((err = hipGetLastError()) != hipSuccess) return err;
    hipLaunchKernelGGL(k_topic_reduce, dim3(uint32_t((p.K + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, d, p, rows, G);
  } else {
    // one wave per region: the workgroup's T table and a count table per wave
    const size_t wlds = sizeof(uint32_t) * (1 + kBlock / kWave) * size_t(p.K);
    err = allow_lds(k_rebuild_w_wave, wlds);
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(k_rebuild_w_wave, dim3(uint32_t(p.grid_regions)), dim3(kBlock), wlds, s, d, p);
  }
  return hipGetLastError();
}

hipError_t launch_rebuild_d(const DevState &d, const Params &p, hipStream_t s) {
  hipError_t err;
  const size_t dlds = sizeof(uint32_t) * d_rebuild_lds_words(p.K) * size_t(p.doc_waves);
  err = allow_lds(k_rebuild_d, dlds);
  if (err != hipSuccess) return err;
  // half the document grid (4 workgroups per CU): fewer waves in flight keep
  // a narrower window of documents, whose topic gathers then hit the caches
  // more often
  const uint32_t dgrid = rebuild_grid(p);
  if (!p.big_k) {
    hipLaunchKernelGGL(k_rebuild_d, dim3(dgrid), dim3(kWave * p.doc_waves), dlds, s, d, p, 1);
    return hipGetLastError();
  }
  // large K: the heavy documents with tables of K counts, the light ones by sorting
  if (p.n_heavy) {
    hipLaunchKernelGGL(k_rebuild_d, dim3(dgrid), dim3(kWave * p.doc_waves), dlds, s, d, p, 0);
    if ((err = hipGetLastError()) != hipSuccess) return err;
  }
  const size_t slds = sizeof(uint16_t) * size_t(kHeavyDoc) * (kBlock / kWave);
  hipLaunchKernelGGL(k_rebuild_d_sort, dim3(uint32_t(p.grid_docs)), dim3(kBlock), slds, s, d, p);
  return hipGetLastError();
}

// ------------------------------------------------- allocation-free LLPT ----
// The scratch of lda_loglik_noalloc: the scheduler counters, the result and
// the per-region partial sums of the LLPT kernels, in one fixed device array
// that every handle on a device shares.  In host code the array's name is not
// a device address: only the address hipGetSymbolAddress returns (one per
// device) may reach a kernel or a copy.
static __device__ __align__(256) unsigned char scratch[kNoAllocHead + sizeof(double) * size_t(LDA_NOALLOC_MAX_REGIONS)];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_addr[kMaxDevices] = {};
}  // namespace

hipError_t noalloc_scratch_address(void **out) {
  *out = nullptr;
  int dev = 0;
  hipError_t err = hipGetDevice(&dev);
  if (err != hipSuccess) return err;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_addr[dev]) {
    void *ptr = nullptr;
    err = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (err != hipSuccess) return err;
    g_scratch_addr[dev] = ptr;
  }
  *out = g_scratch_addr[dev];
  return hipSuccess;
}

hipError_t launch_loglik_noalloc(DevState d, const Params &p, void *scratch_dev, hipStream_t s) {
  if (p.n_regions > int64_t(LDA_NOALLOC_MAX_REGIONS)) return hipErrorInvalidValue;
  unsigned char *base = static_cast<unsigned char *>(scratch_dev);
  d.counters = reinterpret_cast<uint32_t *>(base);                  // cleared by k_begin
  d.ll_out = reinterpret_cast<double *>(base + kNoAllocResult);      // written by k_loglik_reduce
  d.ll_part = reinterpret_cast<double *>(base + kNoAllocHead);       // one slot per region, each written
  d.stats = nullptr;
  hipError_t err = launch_begin_iteration(d, p, s);
  if (err == hipSuccess) err = launch_word_pre(d, p, s);
  if (err == hipSuccess) err = launch_loglik(d, p, s);
  return err;
}

hipError_t launch_sum_f64(const double *part, int64_t n, double *out, hipStream_t s) {
  hipLaunchKernelGGL(k_loglik_reduce, dim3(1), dim3(kBlock), 0, s, part, n, out);
  return hipGetLastError();
}

// The LLPT kernels' dynamic LDS: the W^ row and the batch slices of nb threads.
static size_t loglik_lds_bytes(int K, int nb) {
  return sizeof(double) * (size_t(wh_entries(K)) + size_t(nb) + size_t(nb) / kWave) +
         size_t(nb) * (2 * sizeof(uint32_t) + 1) + 4 * sizeof(uint32_t);
}

int loglik_block(int K) {
  int best = 0, best_waves = 0;
  for (const int nb : {256, 512, 1024}) {
    const int waves = resident_waves(nb == 1024 ? k_loglik_1024 : nb == 512 ? k_loglik_512 : k_loglik, nb, loglik_lds_bytes(K, nb));
    if (waves > best_waves) {
      best = nb;
      best_waves = waves;
    }
  }
  return best;
}

hipError_t launch_loglik(const DevState &d, const Params &p, hipStream_t s) {
  hipError_t err;
  if (p.big_k) {
    // the tile must start at LDS address 0 (wt_of): no static LDS
    static const hipError_t lds_at_0 = no_static_lds(reinterpret_cast<const void *>(k_loglik_tiled));
    if (lds_at_0 != hipSuccess) return lds_at_0;
    const size_t lds = sizeof(double) * (size_t(p.tile_topics) + kGroup + kTiledBlock / kWave) + 4 * sizeof(uint32_t);
    err = allow_lds(k_loglik_tiled, lds);
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(k_loglik_tiled, dim3(uint32_t(tiled_grid(p))), dim3(kTiledBlock), lds, s, d, p);
  } else if (p.n_units > 0) {
    const int nb = p.loglik_block;
    const size_t lds = loglik_lds_bytes(p.K, nb);
    const uint32_t grid = uint32_t(std::min<int64_t>(p.n_units, std::max<int64_t>(1, int64_t(p.grid_regions) * kBlock / nb)));
    if (nb == 1024) {
      err = allow_lds(k_loglik_1024, lds);
      if (err != hipSuccess) return err;
      hipLaunchKernelGGL(k_loglik_1024, dim3(grid), dim3(1024), lds, s, d, p);
    } else if (nb == 512) {
      err = allow_lds(k_loglik_512, lds);
      if (err != hipSuccess) return err;
      hipLaunchKernelGGL(k_loglik_512, dim3(grid), dim3(512), lds, s, d, p);
    } else {
      err = allow_lds(k_loglik, lds);
      if (err != hipSuccess) return err;
      hipLaunchKernelGGL(k_loglik, dim3(grid), dim3(256), lds, s, d, p);
    }
  }
  if ((err = hipGetLastError()) != hipSuccess) return err;
  if (p.n_light_batches > 0) {
    const size_t lds = loglik_lds_bytes(p.K, kWave);
    err = allow_lds(k_loglik_light, lds);
    if (err != hipSuccess) return err;
    const uint32_t grid = uint32_t(light_grid(p));
    hipLaunchKernelGGL(k_loglik_light, dim3(grid), dim3(kWave), lds, s, d, p);
    if ((err = hipGetLastError()) != hipSuccess) return err;
  }
  // one partial per unit and per batch of light regions
  hipLaunchKernelGGL(k_loglik_reduce, dim3(1), dim3(kBlock), 0, s, d.ll_part, p.n_units + p.n_light_batches, d.ll_out);
  return hipGetLastError();
}

}  // namespace lda
