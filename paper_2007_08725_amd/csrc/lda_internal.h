// Internal declarations of liblda: host layout, device state and kernel
// launchers.  Device code targets gfx950 (CDNA4, wave64) only.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>
#include <string>
#include <vector>

#include "../../include/lda.h"

namespace lda {

// Slack entries after the last D row.
constexpr uint32_t kRowPad = 256;

// Slots a D row with nnz entries occupies: its header and entries, rounded
// up to the chunk the sampler reads it in (32 slots up to 128, 64 up to 256,
// then 128).  Every row starts at a multiple of 32 slots (128 bytes), so
// chunks are whole cache lines.  The slots past the entries hold count-0
// entries of topic K (K << 16), whose W^ is 0, so the sampler reads whole
// chunks without bounds checks.
__host__ __device__ inline uint32_t d_row_slots(uint32_t nnz) {
  const uint32_t n = nnz + 1u;
  return n <= 128u ? (n + 31u) & ~31u : n <= 256u ? (n + 63u) & ~63u : (n + 127u) & ~127u;
}
// Words of the per-iteration skip bitmap (one bit per token, a whole number
// of 64-word blocks).
__host__ __device__ inline int64_t skip_words(int64_t n) { return (n + 2047) / 2048 * 64; }
// LDS words (u32) per wave of the D rebuild: K 16-bit counts, a bitmap of K
// bits and a list of up to min(K, 2048) 16-bit topics
__host__ __device__ inline size_t d_rebuild_lds_words(int K) {
  const size_t half = size_t(K + 1) / 2;
  return half + size_t(K + 31) / 32 + (half < 1024 ? half : 1024);
}
constexpr int kDefaultRegionTokens = 10000;  // Sec. 5.1
constexpr int kBlock = 256;                  // threads per workgroup (4 wave64)
constexpr int kXcds = 8;                     // accelerator dies (XCDs), each with its own L2
// Documents longer than this many tokens are heavy: the doc pass and the D
// rebuild give each a whole workgroup instead of a wave (Sec. 5.1).
constexpr uint32_t kHeavyDocTokens = 4096;

// ----------------------------------------------------------------- layout --
// Host-side token layout (Sec. 4.2-4.3 and 5.1).
//   doc order : tokens stably sorted by document
//   word order: tokens stably sorted by relabelled word (within a word the
//               documents ascend, since the source is doc order)
struct Layout {
  int64_t n = 0;
  int32_t M = 0, V = 0, K = 0;
  int32_t n_present = 0;  // words with at least one token (relabelled ids 0..)
  int32_t n_dense = 0;    // relabelled ids [0, n_dense) have count > K
  std::vector<int32_t> relabel;   // [V] caller id -> new id
  std::vector<int32_t> inv;       // [n_present] new id -> caller id
  std::vector<uint32_t> count;    // [n_present] tokens per new id
  std::vector<uint32_t> doc_off;  // [M+1]
  std::vector<uint32_t> word_off; // [n_present+1]
  std::vector<uint32_t> wt_key;   // [n] input index of each word-ordered token (host reference only)
  std::vector<uint32_t> d_cap;    // [M+1] offsets of D rows: a header, then capacity min(len, K)
  std::vector<uint32_t> ws_cap;   // [n_present-n_dense+1] offsets of sparse W rows, capacity = count
  std::vector<uint32_t> region;   // [3*n_regions] (word, begin, end)
  std::vector<uint8_t> split;     // [n_dense] 1 if the dense word has more than one region
  int64_t n_regions = 0;
  int64_t n_dense_regions = 0;
  bool key_identity = false;      // input already doc-sorted: input index == doc-order position
};

// Validates ids (word in [0, V), doc >= 0, n < 2^32); M = max doc + 1 and
// whether the input is already sorted by document.
lda_status scan_tokens(const int32_t *word, const int32_t *doc, int64_t n, int32_t V, int32_t &M, bool &doc_sorted,
                       std::string &msg);
// From the per-word token counts (caller ids) and L.doc_off: relabel, dense
// prefix, relabelled word offsets, capacities and regions.  LDA_E_RANGE for a
// document longer than LDA_MAX_DOC_LEN.
// dense_cutoff as in lda_options (0 = K, negative = all words dense)
// rows = false: relabel, dense prefix and word offsets only (no D and sparse-W
// capacities, no regions: the out-of-core chunks plan their own).
lda_status plan_from_counts(const std::vector<uint32_t> &cnt, int32_t K, int32_t R, int32_t dense_cutoff, Layout &L,
                            std::string &msg, bool rows = true);
// Regions of the words with offsets word_off (Sec. 5.1): words below nd are
// cut into ceil(count / R) regions (split[word] = 1 when more than one), the
// others form one region each, words without tokens none; split words' regions
// first, by the middle of their span, then the rest in word order.
void make_regions(const std::vector<uint32_t> &word_off, int32_t nd, int32_t R, std::vector<uint8_t> &split,
                  std::vector<uint32_t> &region, int64_t &n_dense_regions);
// All-host reference of the layout (lda_describe_layout); fills L.wt_key.
lda_status build_layout(const int32_t *word, const int32_t *doc, int64_t n, int32_t V, int32_t K, int32_t R,
                        int32_t dense_cutoff, Layout &L, std::string &msg);

// Device layout steps (layout_gpu.hip).
unsigned bits_for(uint64_t max_value);
hipError_t sort_pairs_u32(void *tmp, size_t &tmp_bytes, const uint32_t *keys_in, uint32_t *keys_out,
                          const uint32_t *vals_in, uint32_t *vals_out, int64_t n, unsigned end_bit, hipStream_t s);
hipError_t launch_gather_u32(uint32_t *dst, const int32_t *src, const uint32_t *idx, int64_t n, hipStream_t s);
hipError_t launch_boundaries(const uint32_t *keys, int64_t n, uint32_t nbins, uint32_t *off, hipStream_t s);
hipError_t launch_word_order(const uint32_t *wkey, const uint32_t *wpos, int64_t n, const int32_t *relabel,
                             const uint32_t *woff_orig, const uint32_t *woff_new, const uint32_t *doc_sorted,
                             const int32_t *doc_in, const uint32_t *dt_key, uint32_t *dt_word, uint32_t *dt_wpos,
                             const uint32_t *d_cap, uint2 *wt_kr, hipStream_t s);
// bad += topics outside [0, K).
hipError_t launch_check_z(const int32_t *z_in, int64_t n, int32_t K, unsigned long long *bad, hipStream_t s);
hipError_t launch_gather_z(const int32_t *z_in, const uint2 *wt_kr, int64_t n, int32_t K, uint16_t *z_w,
                           unsigned long long *bad, hipStream_t s);
// Out-of-core chunks: the word-order slot of each doc-order position from the
// positions listed in word order; the per-token arrays derived from dt_wpos
// and the chunk's regions and document tables; topics from doc order
// (int32) to word order.
hipError_t launch_invert(const uint32_t *wpos, int64_t n, uint32_t *dt_wpos, hipStream_t s);
hipError_t launch_inflate(const uint32_t *region, int64_t n_regions, const uint32_t *doc_off, const uint32_t *d_cap,
                          int32_t M, const uint32_t *dt_wpos, uint32_t key_base, uint32_t *dt_word, uint2 *wt_kr,
                          hipStream_t s);
hipError_t launch_doc_scatter_z(const int32_t *z_doc, const uint32_t *dt_wpos, int64_t n, int32_t K, uint16_t *z_w,
                                unsigned long long *bad, hipStream_t s);

// ---------------------------------------------------------- device state --
struct WordRec {  // per relabelled word, refreshed every iteration (Sec. 3.2, steps 1 and 4)
  double a1, a2, a3;  // top-3 values of W^[v]
  double qp;          // Q' = sum_{k != K1} alpha * W^[v][k]
  double sumw;        // sum_k W^[v][k] (log-likelihood)
  uint32_t k1, k2;    // top-2 topic ids (lowest id on ties)
};

// Per-word record of the step-3 test in single precision (the test applies a
// margin that covers the rounding, so a skip is always exact).
struct SkipRec {
  uint32_t k12;          // K1 | K2 << 16
  float a1, a2, a3, qp;  // top-3 values of W^[v] and Q' (what the test needs at g <= 2)
  uint32_t k3;           // third top topic (>= K when K < 3)
  float a4;              // fourth top value (g = 3)
  uint32_t pad;
};

struct DevState {
  // layout
  uint32_t *doc_off, *dt_word, *dt_key, *dt_wpos, *word_off;
  uint2 *wt_kr;       // per word-ordered token: (input index = RNG key, D-row offset of its document)
  uint32_t *region;   // 3 per region
  uint32_t *unit;     // 3 per unit of the sampler (sampler_units); the region table itself when no region is cut
  uint32_t *light_batch; // light regions per batch of the light sampler: [n_light_batches + 1], from p.light_begin
  uint32_t *heavy_docs;  // documents longer than kHeavyDoc tokens (one workgroup each in the doc kernels)
  uint8_t *split;     // per dense word
  // assignment, word order
  uint16_t *z_w;
  uint32_t *skip_bits;  // one bit per word-ordered token: the step-3 test drew K1
  uint32_t *skip_doc;   // the same decisions in document order (null when not usable)
  unsigned long long *skip_hist;  // tokens skipped at step 3 by iteration parity: [t & 1]
  // counts
  uint32_t *d_cap, *d_ent;  // D row of doc d at d_cap[d]: header (len << 16 | nnz), then entries
  int32_t *w_dense;
  uint32_t *ws_cap, *ws_nnz, *ws_ent;
  uint32_t *T;
  double *den;
  double *bden;  // beta / den[k]: W^[v][k] where W[v][k] = 0
  WordRec *wrec;
  SkipRec *wskip;
  // scheduler counters and statistics
  uint32_t *counters;           // [kCounters]
  unsigned long long *stats;    // [8]
  unsigned long long *wave_stats; // [kFoldBlocks][kWaveSlots]: per wave of the samplers and the doc pass (StatSlots)
  double *ll_part;              // [n_units + n_light_batches] (large K: [n_regions])
  double *ll_out;               // [1]
  // large K only (k_loglik_tiled): per-workgroup slices of max_region entries
  // carrying a token's sum and split chunk from the first tile to the second
  double *ts_s;
  uint32_t *ts_code;
  uint32_t *hist_rows;  // large K: the rows of k_topic_hist
  // p.sparse_pre: topics by ascending T (descending beta/den[k]),
  // their sort buffers, and [2] the sum of beta/den[k] over all topics with its rounding error
  uint32_t *topic_order, *topic_keys, *topic_iota;
  void *topic_tmp;
  size_t topic_tmp_bytes;
  double *beta_sum;
  double *qbase;  // p.f32: per block of q_block_topics topics the sum of alpha * beta/den[k]
};

struct Params {
  int64_t n;
  int64_t n_all;  // tokens of the whole corpus (n is a chunk's share in the out-of-core mode)
  int32_t M, V, K, n_present, n_dense;
  int64_t n_regions;
  double alpha, beta, vbeta;
  float alpha_f;
  uint64_t seed;
  int32_t g;
  int32_t no_skip;
  int32_t two_branch;  // Sec. 2.2 sampling over [S | Q]: no max-topic branch, no skip test
  int32_t key_identity;
  int32_t grid_regions;  // persistent workgroups for region kernels
  int32_t sampler_block; // threads per sampler workgroup: 256, 512 or 1024
  int32_t grid_docs;     // persistent workgroups for doc kernels
  int32_t big_k;         // the fp64 W^ row does not fit LDS: tiled LLPT, LDS-light rebuilds (K <= 32768)
  int32_t tile_topics;   // topics per tile of k_loglik_tiled (a multiple of 16)
  int32_t max_region;    // tokens of the largest region
  int32_t doc_waves;     // waves per workgroup of the doc pass and the D rebuild (LDS tables of K entries per wave)
  uint32_t doc_batch, rebuild_batch;  // documents a wave takes per counter atomic (doc pass, D rebuild)
  int32_t sparse_pre;    // per-word precompute of sparse words from their row and a topic list (use_topic_list)
  int32_t small_begin;   // sparse words [small_begin, n_present) have at most kSmallWord tokens (with sparse_pre)
  int32_t top_list;      // length of that topic list
  int32_t skip_marks;    // 0 auto, 1 word-ordered bitmap, 2 document-ordered bitmap (lda_options)
  int32_t always_skip_test;  // steps 2-3 every iteration instead of when they pay (lda_options)
  uint32_t key_base;     // out-of-core chunks: input index of the chunk's first doc-ordered token (else 0)
  int32_t n_heavy;       // entries of heavy_docs
  int64_t n_units;       // units of the sampler and the LLPT kernel: the regions before light_begin, cut
  int64_t light_begin;   // regions [light_begin, n_regions): light words, drawn by single waves
  int32_t n_light_batches;  // entries of light_batch, less one
  int32_t doc_marks_ok;  // the document-ordered bitmap is usable: keys are document positions, regular sampler
  int32_t loglik_block;  // threads per workgroup of the LLPT kernel (its W^ row is fp64)
  int32_t f32;           // the sampler keeps W^' in single precision (use_f32)
  int32_t q_table;       // the sampler keeps the Q' blocks' partial sums in LDS (search instead of walk)
  uint32_t xcd_doc[kXcds + 1];  // document ranges with equal token counts, one per XCD (D rebuild)
};

// Workgroups of the D rebuild by tables of K counts (k_rebuild_d) and of the
// doc pass: no more waves than documents (a wave without a document still
// asks every counter), rounded to whole sets of one workgroup per range.
__host__ __device__ inline uint32_t doc_grid(int32_t most, int32_t M, int32_t waves) {
  const int32_t wg = (M + waves - 1) / waves, set = (wg + kXcds - 1) / kXcds * kXcds;
  const int32_t g = set < most ? set : most;
  return uint32_t(g > kXcds ? g : kXcds);
}
inline uint32_t rebuild_grid(const Params &p) { return doc_grid(std::max(1, p.grid_docs / 2), p.M, p.doc_waves); }
__host__ __device__ inline uint32_t doc_pass_grid(const Params &p) { return doc_grid(p.grid_docs, p.M, p.doc_waves); }
// Documents per counter atomic.  Large corpora: 32 in the doc pass and 24 in
// the D rebuild (a smaller window of documents in flight keeps more of its
// topic gathers in the caches).  Small corpora: few enough that every wave of
// the grid gets two batches, down to single documents.
constexpr uint32_t kDocBatch = 32, kRebuildBatch = 24;
inline void set_doc_batches(Params &p) {
  const int64_t w_doc = int64_t(doc_pass_grid(p)) * p.doc_waves, w_reb = int64_t(rebuild_grid(p)) * p.doc_waves;
  p.doc_batch = uint32_t(std::min<int64_t>(kDocBatch, std::max<int64_t>(1, p.M / (2 * w_doc))));
  p.rebuild_batch = uint32_t(std::min<int64_t>(kRebuildBatch, std::max<int64_t>(1, p.M / (2 * w_reb))));
}

// Scheduler counters.  One cache line of the device takes about 88 million
// atomics a second however many addresses in it they go to (8 counters in one
// line 88M/s, in 8 lines 536M/s), so the document kernels' counters, one per
// document range or stripe, sit on lines of their own (kLine words apart);
// the two kernels use different words of them.
constexpr int kLine = 32;  // u32 words per 128-byte line
enum { CNT_SAMPLER = 0, CNT_LOGLIK = 4, CNT_HEAVY_PASS = 5, CNT_HEAVY_REBUILD = 6,
       CNT_DOCPASS = kLine, CNT_REBUILD_D = kLine + 1 };
constexpr int kCounters = kLine * (1 + kXcds);
constexpr int kDocStripes = kXcds;  // counters of the doc pass
enum { ST_SKIP3 = 0, ST_SKIP_AFTER_S = 1, ST_SAMPLED = 2, ST_NNZ = 3, ST_REGIONS = 4, ST_DENSE_REGIONS = 5, ST_ERRORS = 6,
       ST_ROW_BYTES = 7, ST_MARKS = 8, ST_TEST_RAN = 9 };
constexpr int kStatsPerIter = 16;

// The statistics of the samplers and the doc pass: every wave stores its own
// sums and a later launch adds them up.  Atomics on the statistics' one cache
// line cost 55,000 of them, 0.6 ms, an iteration at every corpus size.
enum { WV_SAMPLED, WV_AFTER_S, WV_NNZ, WV_REGIONS, WV_DENSE_REGIONS, WV_ROW_BYTES, WV_SKIP3 };
constexpr int kFoldBlocks = 7;  // one per statistic
constexpr size_t kWaveSlots = size_t(1) << 15;
// Waves that store statistics in iteration t: the main sampler's
// slots come first, then the light sampler's; the doc pass's have a row of
// their own.
struct StatSlots {
  int32_t main, light, doc;  // waves (0: not launched)
  int32_t light0;            // the light sampler's first slot
  uint32_t t;
};

// Kernel launchers (all asynchronous on `s`); return hipGetLastError().
hipError_t launch_init_topics(const DevState &d, const Params &p, hipStream_t s);
hipError_t launch_begin_iteration(const DevState &d, const Params &p, hipStream_t s);
hipError_t launch_word_pre(const DevState &d, const Params &p, hipStream_t s);
hipError_t launch_beta_sum(const DevState &d, const Params &p, hipStream_t s);
// reset_count: also clear this iteration's skip count (false for the second
// and later chunks of an out-of-core iteration, which add to it)
hipError_t launch_clear_skips(const DevState &d, const Params &p, uint32_t t, hipStream_t s, bool reset_count = true);
hipError_t launch_reset_counters(uint32_t *counters, hipStream_t s);
hipError_t launch_doc_pass(const DevState &d, const Params &p, uint32_t t, hipStream_t s);
// The sampler of the regions before p.light_begin, and that of the light regions, by single waves (nothing when
// there are none); the two touch disjoint topic slots and may run at once.
hipError_t launch_sampler(const DevState &d, const Params &p, uint32_t t, hipStream_t s);
hipError_t launch_sampler_light(const DevState &d, const Params &p, uint32_t t, hipStream_t s);
bool sampler_q_table(int K);
// The sampler that keeps W^' in single precision and certifies its draws:
// topics per block of its Q' prefix, its workgroup size and dynamic LDS, and
// the K it is used from: where the fp64 row starts to limit the resident
// waves (22.8 KB a workgroup for 7 workgroups per CU).  Below, the fp64 one is
// as fast or faster (144M tokens at K = 1,000: 7.66 ms, the other 7.87), above
// not (33M at K = 10,000: 9.8 against 6.7 ms; 20M at 32,768, where fp64 took
// the row in two tiles: 15.8 against 8.7).  Workgroups of 512 and 1,024
// threads (an option) are its own at every K.
// (16 with 256 threads, where the LDS has room for K / 16 doubles, else 32)
__host__ __device__ constexpr int q_block_topics(int threads) { return threads == 256 ? 16 : 32; }
constexpr int kF32Topics = 2300;
inline bool use_f32(int32_t K, int32_t want_block) { return K >= kF32Topics || (want_block != 0 && want_block != kBlock); }
// Its bounds (why they hold: kernels.hip, "certified draws").  S' and its
// prefixes are off by at most kEps of S; S here is S' rounded up, tau covers
// the fp64 roundings and underflow; M is any number not below the max-topic
// branch.  s_bound: x against M and against the edges inside S'.  q_bound: x
// less M + S'.  q_bound_f: the same inside a Q' block of bs topics walked in
// fp32, in units of alpha * 2^-24 (inv of them to 1): x rounded once, at most
// bs + 1 roundings in a partial sum, two more in the comparison; p is the sum
// of the block.
constexpr double kEps = 9.5 * 0x1p-24;
constexpr double kWScale = 0x1p24;  // the row holds W^' * 2^24
__host__ __device__ inline double draw_tau(double M, double S, double qp) { return (M + S + qp) * 0x1p-40 + 0x1p-90; }
__host__ __device__ inline double s_bound(double S, double tau) { return 2.0 * kEps * S + tau; }
__host__ __device__ inline double q_bound(double S, double qp, double tau) {
  return kEps * S * (qp / (S + qp)) * (1.0 + 0x1p-20) + tau;
}
__host__ __device__ inline float q_bound_f(double eq, float inv, float p, float xb, int bs) {
  return float(eq) * inv * (1.0f + 0x1p-20f) + (p + xb) * (float(bs + 4) * 0x1p-24f);
}
// Its Q' block sums are added up by many lanes in no fixed order, so they are
// whole numbers of units of 2^(ex - 62), 2^ex being the power of two above the
// word's Q': any order gives the same bits, no sum passes 2^62 by more than
// the terms' roundings, and a term is off by at most 2^-62 of Q' (an fp64 sum
// by 2^-53 of itself at each addition).  The terms are the block's sum of
// alpha * beta/den[k] (K1's block: of the other topics) and
// alpha * (W^[v][k] - beta/den[k]) of every topic that the word holds.
__host__ __device__ inline int q_exponent(double qp) {
  int ex = 0;
  (void)frexp(qp, &ex);
  return ex;
}
__host__ __device__ inline unsigned long long q_units(double v, int ex) {
  return (unsigned long long)rint(ldexp(v, 62 - ex));
}
__host__ __device__ inline double q_value(unsigned long long units, int ex) {
  return ldexp(double(units), ex - 62);
}
int sampler_f_block(int K, int want);
size_t sampler_f_lds_bytes(int K, int nb);
int loglik_block(int K);  // threads per workgroup of k_loglik (the most resident waves)
// The sampler's dynamic LDS for K topics and workgroups of nb threads.
size_t sampler_lds_bytes(int K, int nb, bool q_table);
// Regions of at most this many tokens (one batch of the sampler) are light:
// single waves take them, several words at a time, when the per-wave W^' row
// is small (K up to about 2,200: 8 waves per CU, against as many workgroups of
// the regular sampler).  They form a suffix of the region table, which lists
// the unsplit words by descending token count after the split ones.
constexpr uint32_t kLightTokens = 64;
constexpr size_t kLightLdsMax = 20 * 1024;
size_t light_lds_bytes(int K);
inline int64_t light_region_start(const std::vector<uint32_t> &region, int K, bool big_k) {
  int64_t r = int64_t(region.size() / 3);
  if (big_k || light_lds_bytes(K) > kLightLdsMax) return r;
  while (r > 0 && region[3 * size_t(r - 1) + 2] - region[3 * size_t(r - 1) + 1] <= kLightTokens) --r;
  return r;
}
// The regions before light_begin cut into the units that workgroups of the
// sampler take, in the regions' order: (word, begin, end), bit 31 of the word
// set in a unit that continues a region.  A region of up to 10,000 tokens keeps
// one workgroup busy for a hundred batches, so a small corpus is cut finer:
// into about two units per resident workgroup, but not below the tokens that
// give every wave a batch, nor below twice the K topics that a unit's W^ row
// costs (50,000 tokens at K = 16: sampler 0.146 -> 0.045 ms, 610,000 at K = 101
// 0.324 -> 0.131; four units instead of two, or a least unit of K / 2, cost 9M
// tokens at K = 2,000 10%).  Draws do not depend on the cut.
constexpr uint32_t kUnitContinues = 0x80000000u;
std::vector<uint32_t> sampler_units(const std::vector<uint32_t> &region, int64_t light_begin, int64_t n, int32_t K,
                                    int64_t workgroups, int32_t threads);
__host__ __device__ inline int64_t sampler_workgroups(const Params &p) {
  const int64_t w = int64_t(p.grid_regions) * kBlock / (p.sampler_block > 0 ? p.sampler_block : kBlock);
  return w > 0 ? w : 1;
}
// The light regions cut into batches of consecutive word-ordered tokens, as
// offsets from light_begin: at most 64 tokens each, fewer (down to 16) when
// that would leave the light sampler's waves without a batch.
std::vector<uint32_t> light_batches(const std::vector<uint32_t> &region, int64_t light_begin, int64_t waves);
// Large K: topics per tile of k_loglik_tiled.
int tiled_topics(int K);
// Workgroups of k_loglik_tiled (one per CU: its LDS fills a CU) and of
// k_topic_hist; the scratch slices are sized for these grids.
__host__ __device__ inline int tiled_grid(const Params &p) { return p.grid_regions / 8 > 0 ? p.grid_regions / 8 : 1; }
inline int topic_hist_grid(const Params &p) { return tiled_grid(p); }
// Workgroups of the main and of the light sampler (at most 16
// one-wave workgroups per CU; grid_regions is 8 per CU), and the statistics
// slots of an iteration's launches.
__host__ __device__ inline int32_t sampler_grid(const Params &p) {
  const int64_t w = sampler_workgroups(p);
  return int32_t(p.n_units < w ? p.n_units : w);
}
__host__ __device__ inline int32_t light_grid(const Params &p) {
  return p.n_light_batches < 2 * p.grid_regions ? p.n_light_batches : 2 * p.grid_regions;
}
__host__ __device__ inline StatSlots stat_slots(const Params &p, uint32_t t) {
  StatSlots s;
  s.main = sampler_grid(p) * (p.sampler_block / 64);
  s.light0 = s.main;
  s.light = light_grid(p);
  s.doc = p.no_skip ? 0 : int32_t(doc_pass_grid(p)) * p.doc_waves;
  s.t = t;
  return s;
}
// Whether every launch's waves have a slot (grids follow the device's CUs).
inline bool stat_slots_fit(const Params &p) {
  const int64_t main = sampler_workgroups(p);
  return main * (p.sampler_block / 64) + 2 * int64_t(p.grid_regions) <= int64_t(kWaveSlots) &&
         int64_t(std::max(p.grid_docs, kXcds)) * p.doc_waves <= int64_t(kWaveSlots);
}
// The W rebuild by bitmap, with T from a histogram of the topics (and its
// scratch rows), from this many topics on: below it a workgroup's tables of K
// counts are small enough to keep several workgroups on a CU.
constexpr int kWBitsK = 4096;
// The per-word precompute of sparse words from their rows and a list of the
// topics with the largest beta/den[k], instead of K topics per word: from
// K = 4,096 on, where a wave's table of K counts gets large, and below it when
// the sparse words' tables would be at least 4M topics together (about 40 us;
// the list is a launch of its own, 6 us at K = 1,000).
// The list is in the order of T; the top topics are by beta/den[k], the lowest
// id first among equals.  The two orders are the same while beta/den[k] differs
// wherever T does: den = T + V*beta below 2^50 (neighbours then differ by three
// units in the last place of the quotient) and no quotient near underflow.
// With priors beyond, every topic is looked at: by tables of counts below
// K = 4,096, from there on by searches of the row (a list of no topics).
constexpr uint32_t kSmallWord = 64;
inline bool topic_list_ordered(double beta, double vbeta, int64_t n) {
  return vbeta + double(n) < 0x1p50 && beta > 0x1p-960;
}
inline bool use_topic_list(int32_t K, int64_t sparse_words, bool ordered) {
  return K >= kWBitsK || (ordered && sparse_words * K >= (int64_t(4) << 20));
}
inline bool w_bits(const Params &p) { return p.big_k || p.K >= kWBitsK; }
// The count rebuild (Sec. 4.3): launch_rebuild = launch_zero_split, then
// launch_rebuild_w and launch_rebuild_d.
// slots: also add up the statistics of the samplers and the doc pass that ran.
hipError_t launch_rebuild(const DevState &d, const Params &p, hipStream_t s, const StatSlots *slots = nullptr);
hipError_t launch_zero_split(const DevState &d, const Params &p, hipStream_t s, const StatSlots *slots = nullptr);
hipError_t launch_fold_stats(const DevState &d, const StatSlots &slots, hipStream_t s);
hipError_t launch_rebuild_w(const DevState &d, const Params &p, hipStream_t s);
hipError_t launch_rebuild_d(const DevState &d, const Params &p, hipStream_t s);
hipError_t launch_loglik(const DevState &d, const Params &p, hipStream_t s);
// out[0] = sum of part[0..n) in a fixed order (one workgroup).
hipError_t launch_sum_f64(const double *part, int64_t n, double *out, hipStream_t s);
// Allocation-free LLPT: the layout of the fixed scratch array (counters at 0,
// the result at kNoAllocResult, out-of-core per-chunk sums at
// kNoAllocChunkSums, per-region partials from kNoAllocHead), its
// device address on the current device (looked up once per device), and the
// LLPT launches on it.  hipErrorInvalidValue past LDA_NOALLOC_MAX_REGIONS.
constexpr size_t kNoAllocResult = 1536;
constexpr size_t kNoAllocChunkSums = 2048;
constexpr size_t kNoAllocHead = 4096;
static_assert(kNoAllocChunkSums + sizeof(double) * LDA_MAX_CHUNKS <= kNoAllocHead, "chunk sums overlap the partials");
static_assert(sizeof(uint32_t) * kCounters + sizeof(unsigned long long) * kStatsPerIter <= kNoAllocResult,
              "counters and statistics overlap the result");
hipError_t noalloc_scratch_address(void **out);
hipError_t launch_loglik_noalloc(DevState d, const Params &p, void *scratch_dev, hipStream_t s);
// Exports of lda_get_counts.  out[0] += entries of the D rows, out[1] +=
// entries of W (either may be left out); the topics in doc order or, with
// dt_key (input not sorted by document), in input order; entries per document
// and per relabelled word; D entries and W (topic, count) pairs of a slab of
// rows compacted at off[] (relative to the slab).
hipError_t launch_sum_nnz(const DevState &d, const Params &p, bool D, bool W, unsigned long long *out, hipStream_t s);
hipError_t launch_gather_z16(const uint32_t *dt_wpos, const uint32_t *dt_key, const uint16_t *z_w, int64_t n,
                             uint16_t *z_out, hipStream_t s);
hipError_t launch_doc_nnz(const DevState &d, int64_t doc0, int64_t n, uint32_t *num, hipStream_t s);
hipError_t launch_word_nnz(const DevState &d, const Params &p, uint32_t *num, hipStream_t s);
hipError_t launch_export_d(const DevState &d, int64_t doc0, int64_t n, const uint32_t *off, uint32_t *out,
                           hipStream_t s);
hipError_t launch_export_w(const DevState &d, const Params &p, const uint32_t *row, const uint32_t *off, int64_t n,
                           uint2 *out, hipStream_t s);

}  // namespace lda
