// Token layout on the device (lda_create): the two stable orders of Sec. 4.3
// built with rocPRIM radix sorts, plus the gathers/scatters that link them.
//
//   doc order : stable sort of input indices by document (skipped when the
//               input is already sorted by document)
//   word order: stable sort of doc-order positions by caller word id, then a
//               permutation of whole word segments into relabelled order
//               (descending count, Sec. 4.2), so that within a word the
//               documents ascend.
#include <rocprim/device/device_radix_sort.hpp>
#include <rocprim/iterator/counting_iterator.hpp>

#include "lda_internal.h"

namespace lda {
namespace {

constexpr int kThreads = 256;

inline uint32_t grid_for(int64_t n) {
  const int64_t b = (n + kThreads - 1) / kThreads;
  return uint32_t(std::min<int64_t>(std::max<int64_t>(b, 1), 1 << 20));
}

__global__ void k_gather_u32(uint32_t *__restrict__ dst, const int32_t *__restrict__ src,
                             const uint32_t *__restrict__ idx, int64_t n) {
  for (int64_t p = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; p < n; p += int64_t(gridDim.x) * blockDim.x)
    dst[p] = uint32_t(src[idx[p]]);
}

// off[b] = first position whose key is >= b, for b in [0, nbins]; keys ascending.
__global__ void k_boundaries(const uint32_t *__restrict__ keys, int64_t n, uint32_t nbins, uint32_t *__restrict__ off) {
  for (int64_t p = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; p < n; p += int64_t(gridDim.x) * blockDim.x) {
    const uint32_t k = keys[p];
    const int64_t prev = p == 0 ? -1 : int64_t(keys[p - 1]);
    for (int64_t b = prev + 1; b <= int64_t(k); ++b) off[b] = uint32_t(p);
    if (p == n - 1)
      for (int64_t b = int64_t(k) + 1; b <= int64_t(nbins); ++b) off[b] = uint32_t(n);
  }
}

// Word-order slot of every token: its position in the caller-id sort, moved
// with its whole word segment to the relabelled segment start.  Each
// word-ordered token records the offset of its document's D row.
__global__ void k_word_order(const uint32_t *__restrict__ wkey, const uint32_t *__restrict__ wpos, int64_t n,
                             const int32_t *__restrict__ relabel, const uint32_t *__restrict__ woff_orig,
                             const uint32_t *__restrict__ woff_new, const uint32_t *__restrict__ doc_sorted,
                             const int32_t *__restrict__ doc_in, const uint32_t *__restrict__ dt_key,
                             uint32_t *__restrict__ dt_word, uint32_t *__restrict__ dt_wpos,
                             const uint32_t *__restrict__ d_cap, uint2 *__restrict__ wt_kr) {
  for (int64_t q = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; q < n; q += int64_t(gridDim.x) * blockDim.x) {
    const uint32_t v = wkey[q];
    const uint32_t r = uint32_t(relabel[v]);
    const uint32_t j = woff_new[r] + (uint32_t(q) - woff_orig[v]);
    const uint32_t p = wpos[q];
    dt_word[p] = r;
    dt_wpos[p] = j;
    wt_kr[j] = make_uint2(dt_key ? dt_key[p] : p, d_cap[doc_sorted ? doc_sorted[p] : uint32_t(doc_in[p])]);
  }
}

__global__ void k_check_z(const int32_t *__restrict__ z, int64_t n, int32_t K, unsigned long long *__restrict__ bad) {
  unsigned long long nbad = 0;
  for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += int64_t(gridDim.x) * blockDim.x)
    nbad += z[i] < 0 || z[i] >= K ? 1ull : 0ull;
  if (nbad) atomicAdd(bad, nbad);
}

__global__ void k_gather_z(const int32_t *__restrict__ z_in, const uint2 *__restrict__ wt_kr, int64_t n,
                           int32_t K, uint16_t *__restrict__ z_w, unsigned long long *__restrict__ bad) {
  unsigned long long nbad = 0;
  for (int64_t j = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; j < n; j += int64_t(gridDim.x) * blockDim.x) {
    const int32_t z = z_in[wt_kr[j].x];
    if (z >= 0 && z < K) z_w[j] = uint16_t(z);
    else {
      z_w[j] = 0;
      nbad++;
    }
  }
  if (nbad) atomicAdd(bad, nbad);
}

// ----------------------------------------------------- out-of-core chunks --
// A chunk keeps only dt_wpos (word-order slot of each doc-ordered token) and
// its topics in host memory; the other per-token arrays are derived on the
// device when the chunk is loaded.

// dt_wpos[wpos[q]] = q: the word-order slot of each doc-order position, from
// the doc-order positions listed in word order.
__global__ void k_invert(const uint32_t *__restrict__ wpos, int64_t n, uint32_t *__restrict__ dt_wpos) {
  for (int64_t q = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; q < n; q += int64_t(gridDim.x) * blockDim.x)
    dt_wpos[wpos[q]] = uint32_t(q);
}

// slot_word[s] = the word of word-order slot s, one workgroup per region
// (the regions cover every slot exactly once).
__global__ void k_slot_words(const uint32_t *__restrict__ region, int64_t n_regions, uint2 *__restrict__ wt_kr) {
  for (int64_t r = blockIdx.x; r < n_regions; r += gridDim.x) {
    const uint32_t v = region[3 * r], b = region[3 * r + 1], e = region[3 * r + 2];
    for (uint32_t s = b + threadIdx.x; s < e; s += blockDim.x) wt_kr[s] = make_uint2(0u, v);
  }
}

// Per document, one wave: for each of its tokens p (slot s = dt_wpos[p]) the
// word id in doc order, and the key (key_base + p, the input index: chunks
// need input sorted by document) and D-row offset in word order.  The word of
// slot s (k_slot_words) waits in the second half of its (key, row offset)
// record, which the one token that owns the slot reads and then overwrites:
// one scattered 8-byte record per token, read and written in the same line.
__global__ void k_inflate(const uint32_t *__restrict__ doc_off, const uint32_t *__restrict__ d_cap, int32_t M,
                          const uint32_t *__restrict__ dt_wpos, uint32_t key_base, uint32_t *__restrict__ dt_word,
                          uint2 *__restrict__ wt_kr) {
  const int lane = threadIdx.x & 63, waves = int(blockDim.x) / 64;
  for (int64_t d = int64_t(blockIdx.x) * waves + threadIdx.x / 64; d < M; d += int64_t(gridDim.x) * waves) {
    const uint32_t b = doc_off[d], e = doc_off[d + 1], cap = d_cap[d];
    for (uint32_t p = b + uint32_t(lane); p < e; p += 64u) {
      const uint32_t s = dt_wpos[p];
      dt_word[p] = wt_kr[s].y;
      wt_kr[s] = make_uint2(key_base + p, cap);
    }
  }
}

// Topics in word order from topics in doc order (int32), with a range check
// (bad counts topics outside [0, K), which are stored as 0).
__global__ void k_doc_scatter_z(const int32_t *__restrict__ z_doc, const uint32_t *__restrict__ dt_wpos, int64_t n,
                                int32_t K, uint16_t *__restrict__ z_w, unsigned long long *__restrict__ bad) {
  unsigned long long nbad = 0;
  for (int64_t p = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; p < n; p += int64_t(gridDim.x) * blockDim.x) {
    const int32_t z = z_doc[p];
    const bool ok = z >= 0 && z < K;
    z_w[dt_wpos[p]] = ok ? uint16_t(z) : uint16_t(0);
    nbad += ok ? 0ull : 1ull;
  }
  if (nbad) atomicAdd(bad, nbad);
}

// ----------------------------------------------------------------- exports --
// The kernels of lda_get_counts.  All are bound by memory (each table is read
// once); what they replace is the tables' way over PCIe: the dense rows of W
// were copied to the host to count their entries (564 MB, 158 ms a call, for
// 141,000 out-of-core words at K = 1,000), and rows were walked by one host
// thread.

__global__ void k_gather_z16(const uint32_t *__restrict__ dt_wpos, const uint32_t *__restrict__ dt_key,
                             const uint16_t *__restrict__ z_w, int64_t n, uint16_t *__restrict__ z_out) {
  for (int64_t p = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; p < n; p += int64_t(gridDim.x) * blockDim.x)
    z_out[dt_key ? dt_key[p] : uint32_t(p)] = z_w[dt_wpos[p]];
}

__device__ __forceinline__ unsigned long long wave_total(unsigned long long v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

__global__ __launch_bounds__(kThreads) void k_sum_nnz(DevState d, Params p, int D, int W,
                                                      unsigned long long *__restrict__ out) {
  const int64_t i0 = int64_t(blockIdx.x) * blockDim.x + threadIdx.x, step = int64_t(gridDim.x) * blockDim.x;
  unsigned long long nd = 0, nw = 0;
  if (D)
    for (int64_t q = i0; q < p.M; q += step) nd += d.d_ent[d.d_cap[q]] & 0xFFFFu;
  if (W) {
    // the dense table by 16 bytes (global loads of 16 bytes need 4-byte alignment only), then its last values
    const int64_t total = int64_t(p.n_dense) * p.K, quads = total / 4;
    const int4 *w4 = reinterpret_cast<const int4 *>(d.w_dense);
    for (int64_t q = i0; q < quads; q += step) {
      const int4 v = w4[q];
      nw += uint32_t(v.x != 0) + uint32_t(v.y != 0) + uint32_t(v.z != 0) + uint32_t(v.w != 0);
    }
    if (quads * 4 + i0 < total) nw += d.w_dense[quads * 4 + i0] != 0;
    for (int64_t q = i0; q < p.n_present - p.n_dense; q += step) nw += d.ws_nnz[q];
  }
  // one atomic per workgroup and sum: a cache line takes 88 million a second
  __shared__ unsigned long long s_sum[2][kThreads / 64];
  nd = wave_total(nd);
  nw = wave_total(nw);
  if ((threadIdx.x & 63) == 0) {
    s_sum[0][threadIdx.x / 64] = nd;
    s_sum[1][threadIdx.x / 64] = nw;
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    unsigned long long v = 0;
    for (int q = 0; q < kThreads / 64; ++q) v += s_sum[threadIdx.x][q];
    if (v) atomicAdd(&out[threadIdx.x], v);
  }
}

__global__ void k_doc_nnz(DevState d, int64_t doc0, int64_t n, uint32_t *__restrict__ num) {
  for (int64_t q = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; q < n; q += int64_t(gridDim.x) * blockDim.x)
    num[q] = d.d_ent[d.d_cap[doc0 + q]] & 0xFFFFu;
}

// One wave per word.
__global__ __launch_bounds__(kThreads) void k_word_nnz(DevState d, Params p, uint32_t *__restrict__ num) {
  const int lane = threadIdx.x & 63;
  for (int64_t r = int64_t(blockIdx.x) * (kThreads / 64) + threadIdx.x / 64; r < p.n_present;
       r += int64_t(gridDim.x) * (kThreads / 64)) {
    if (r >= p.n_dense) {
      if (lane == 0) num[r] = d.ws_nnz[r - p.n_dense];
      continue;
    }
    const int32_t *row = d.w_dense + size_t(r) * size_t(p.K);
    uint32_t c = 0;
    for (int k = lane; k < p.K; k += 64) c += row[k] != 0;
    c = uint32_t(wave_total(c));
    if (lane == 0) num[r] = c;
  }
}

// 16 lanes per document.
__global__ void k_export_d(DevState d, int64_t doc0, int64_t n, const uint32_t *__restrict__ off,
                           uint32_t *__restrict__ out) {
  const int li = threadIdx.x & 15;
  for (int64_t q = int64_t(blockIdx.x) * (kThreads / 16) + threadIdx.x / 16; q < n;
       q += int64_t(gridDim.x) * (kThreads / 16)) {
    const uint32_t *row = d.d_ent + d.d_cap[doc0 + q];
    const uint32_t m = row[0] & 0xFFFFu, o = off[q];
    for (uint32_t i = uint32_t(li); i < m; i += 16u) out[o + i] = row[1u + i];
  }
}

// One wave per word: a dense row's nonzero counts compacted by ballot, a
// sparse row's entries unpacked.
__global__ __launch_bounds__(kThreads) void k_export_w(DevState d, Params p, const uint32_t *__restrict__ row,
                                                       const uint32_t *__restrict__ off, int64_t n,
                                                       uint2 *__restrict__ out) {
  const int lane = threadIdx.x & 63;
  for (int64_t i = int64_t(blockIdx.x) * (kThreads / 64) + threadIdx.x / 64; i < n;
       i += int64_t(gridDim.x) * (kThreads / 64)) {
    const uint32_t r = row[i];
    uint32_t o = off[i];
    if (r < uint32_t(p.n_dense)) {
      const int32_t *w = d.w_dense + size_t(r) * size_t(p.K);
      for (int k0 = 0; k0 < p.K; k0 += 64) {
        const int k = k0 + lane;
        const int32_t c = k < p.K ? w[k] : 0;
        const unsigned long long m = __ballot(c != 0);
        const uint32_t rank = __builtin_amdgcn_mbcnt_hi(uint32_t(m >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(m), 0u));
        if (c != 0) out[o + rank] = make_uint2(uint32_t(k), uint32_t(c));
        o += uint32_t(__popcll(m));
      }
    } else {
      const uint32_t s = r - uint32_t(p.n_dense), m = d.ws_nnz[s];
      const uint32_t *e = d.ws_ent + d.ws_cap[s];
      for (uint32_t q = uint32_t(lane); q < m; q += 64u) out[o + q] = make_uint2(e[q] >> 16, e[q] & 0xFFFFu);
    }
  }
}

}  // namespace

hipError_t launch_invert(const uint32_t *wpos, int64_t n, uint32_t *dt_wpos, hipStream_t s) {
  hipLaunchKernelGGL(k_invert, dim3(grid_for(n)), dim3(kThreads), 0, s, wpos, n, dt_wpos);
  return hipGetLastError();
}

hipError_t launch_inflate(const uint32_t *region, int64_t n_regions, const uint32_t *doc_off, const uint32_t *d_cap,
                          int32_t M, const uint32_t *dt_wpos, uint32_t key_base, uint32_t *dt_word, uint2 *wt_kr,
                          hipStream_t s) {
  const uint32_t rg = uint32_t(std::min<int64_t>(std::max<int64_t>(n_regions, 1), 1 << 16));
  hipLaunchKernelGGL(k_slot_words, dim3(rg), dim3(kThreads), 0, s, region, n_regions, wt_kr);
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  const int64_t waves = kThreads / 64;
  const uint32_t dg = uint32_t(std::min<int64_t>(std::max<int64_t>((int64_t(M) + waves - 1) / waves, 1), 1 << 16));
  hipLaunchKernelGGL(k_inflate, dim3(dg), dim3(kThreads), 0, s, doc_off, d_cap, M, dt_wpos, key_base, dt_word, wt_kr);
  return hipGetLastError();
}

hipError_t launch_sum_nnz(const DevState &d, const Params &p, bool D, bool W, unsigned long long *out, hipStream_t s) {
  const int64_t work = std::max<int64_t>(D ? p.M : 0, W ? std::max<int64_t>(int64_t(p.n_dense) * p.K / 16, p.n_present) : 0);
  const uint32_t grid = std::min(grid_for(work), 1024u);
  hipLaunchKernelGGL(k_sum_nnz, dim3(grid), dim3(kThreads), 0, s, d, p, D ? 1 : 0, W ? 1 : 0, out);
  return hipGetLastError();
}

hipError_t launch_gather_z16(const uint32_t *dt_wpos, const uint32_t *dt_key, const uint16_t *z_w, int64_t n,
                             uint16_t *z_out, hipStream_t s) {
  hipLaunchKernelGGL(k_gather_z16, dim3(grid_for(n)), dim3(kThreads), 0, s, dt_wpos, dt_key, z_w, n, z_out);
  return hipGetLastError();
}

hipError_t launch_doc_nnz(const DevState &d, int64_t doc0, int64_t n, uint32_t *num, hipStream_t s) {
  hipLaunchKernelGGL(k_doc_nnz, dim3(grid_for(n)), dim3(kThreads), 0, s, d, doc0, n, num);
  return hipGetLastError();
}

hipError_t launch_word_nnz(const DevState &d, const Params &p, uint32_t *num, hipStream_t s) {
  hipLaunchKernelGGL(k_word_nnz, dim3(grid_for(int64_t(p.n_present) * 64)), dim3(kThreads), 0, s, d, p, num);
  return hipGetLastError();
}

hipError_t launch_export_d(const DevState &d, int64_t doc0, int64_t n, const uint32_t *off, uint32_t *out,
                           hipStream_t s) {
  hipLaunchKernelGGL(k_export_d, dim3(grid_for(n * 16)), dim3(kThreads), 0, s, d, doc0, n, off, out);
  return hipGetLastError();
}

hipError_t launch_export_w(const DevState &d, const Params &p, const uint32_t *row, const uint32_t *off, int64_t n,
                           uint2 *out, hipStream_t s) {
  hipLaunchKernelGGL(k_export_w, dim3(grid_for(n * 64)), dim3(kThreads), 0, s, d, p, row, off, n, out);
  return hipGetLastError();
}

hipError_t launch_doc_scatter_z(const int32_t *z_doc, const uint32_t *dt_wpos, int64_t n, int32_t K, uint16_t *z_w,
                                unsigned long long *bad, hipStream_t s) {
  hipLaunchKernelGGL(k_doc_scatter_z, dim3(grid_for(n)), dim3(kThreads), 0, s, z_doc, dt_wpos, n, K, z_w, bad);
  return hipGetLastError();
}

unsigned bits_for(uint64_t max_value) {
  unsigned b = 1;
  while (b < 32 && (max_value >> b)) ++b;
  return b;
}

hipError_t sort_pairs_u32(void *tmp, size_t &tmp_bytes, const uint32_t *keys_in, uint32_t *keys_out,
                          const uint32_t *vals_in, uint32_t *vals_out, int64_t n, unsigned end_bit, hipStream_t s) {
  const size_t size = size_t(n);
  if (vals_in)
    return rocprim::radix_sort_pairs(tmp, tmp_bytes, keys_in, keys_out, vals_in, vals_out, size, 0u, end_bit, s);
  return rocprim::radix_sort_pairs(tmp, tmp_bytes, keys_in, keys_out, rocprim::counting_iterator<uint32_t>(0u),
                                   vals_out, size, 0u, end_bit, s);
}

hipError_t launch_gather_u32(uint32_t *dst, const int32_t *src, const uint32_t *idx, int64_t n, hipStream_t s) {
  hipLaunchKernelGGL(k_gather_u32, dim3(grid_for(n)), dim3(kThreads), 0, s, dst, src, idx, n);
  return hipGetLastError();
}

hipError_t launch_boundaries(const uint32_t *keys, int64_t n, uint32_t nbins, uint32_t *off, hipStream_t s) {
  hipLaunchKernelGGL(k_boundaries, dim3(grid_for(n)), dim3(kThreads), 0, s, keys, n, nbins, off);
  return hipGetLastError();
}

hipError_t launch_word_order(const uint32_t *wkey, const uint32_t *wpos, int64_t n, const int32_t *relabel,
                             const uint32_t *woff_orig, const uint32_t *woff_new, const uint32_t *doc_sorted,
                             const int32_t *doc_in, const uint32_t *dt_key, uint32_t *dt_word, uint32_t *dt_wpos,
                             const uint32_t *d_cap, uint2 *wt_kr, hipStream_t s) {
  hipLaunchKernelGGL(k_word_order, dim3(grid_for(n)), dim3(kThreads), 0, s, wkey, wpos, n, relabel, woff_orig,
                     woff_new, doc_sorted, doc_in, dt_key, dt_word, dt_wpos, d_cap, wt_kr);
  return hipGetLastError();
}

hipError_t launch_check_z(const int32_t *z_in, int64_t n, int32_t K, unsigned long long *bad, hipStream_t s) {
  hipLaunchKernelGGL(k_check_z, dim3(std::min(grid_for(n), 4096u)), dim3(kThreads), 0, s, z_in, n, K, bad);
  return hipGetLastError();
}

hipError_t launch_gather_z(const int32_t *z_in, const uint2 *wt_kr, int64_t n, int32_t K, uint16_t *z_w,
                           unsigned long long *bad, hipStream_t s) {
  hipLaunchKernelGGL(k_gather_z, dim3(grid_for(n)), dim3(kThreads), 0, s, z_in, wt_kr, n, K, z_w, bad);
  return hipGetLastError();
}

}  // namespace lda
