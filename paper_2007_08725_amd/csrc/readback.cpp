// Exports of lda_get_counts: the count tables are compacted to CSR on the
// device, a bounded slab of rows at a time, and read back through the handle's
// pinned buffers (readback.h).
#include "readback.h"

namespace lda {

namespace {
constexpr size_t kSlabEntries = size_t(1) << 23;  // entries of a slab (32 MB of D entries, 64 MB of W pairs)
constexpr size_t kSlabRows = size_t(1) << 21;     // rows of a slab
}  // namespace

namespace {
auto widen_to(int32_t *out) {
  return [out](const uint16_t *src, size_t first, size_t m) {
    int32_t *dst = out + first;
    for (size_t i = 0; i < m; ++i) dst[i] = int32_t(src[i]);
  };
}
}  // namespace

lda_status read_z(lda_handle *h, Crew &crew, const uint16_t *z, size_t n, int32_t *out) {
  return read_back(h, crew, z, n, widen_to(out));
}
lda_status read_z(lda_handle *h, Crew &crew, const Scratch<uint16_t> &z, size_t n, int32_t *out) {
  return read_back(h, crew, z, n, widen_to(out));
}

lda_status export_d(lda_handle *h, Crew &crew, const DevState &d, int32_t M, int64_t at, int64_t *off, int32_t *topic,
                    int32_t *count, int64_t *entries) {
  *entries = 0;
  const size_t docs = size_t(M), rows = std::min(docs, kSlabRows);
  if (!docs) {
    off[0] = at;
    return LDA_OK;
  }
  Scratch<uint32_t> num(h), ent(h);
  LDA_TRY(num.get(rows));
  std::vector<uint32_t> n(docs);
  for (size_t a = 0; a < docs; a += rows) {
    const size_t m = std::min(rows, docs - a);
    HIP_TRY(h, launch_doc_nnz(d, int64_t(a), int64_t(m), num.ptr, h->stream));
    LDA_TRY(read_back(h, crew, num, m, [&](const uint32_t *src, size_t first, size_t k) {
      std::memcpy(n.data() + a + first, src, k * sizeof(uint32_t));
    }));
  }
  int64_t o = at;
  for (size_t q = 0; q < docs; ++q) {
    off[q] = o;
    o += n[q];
  }
  off[docs] = o;
  *entries = o - at;
  // a row has fewer than 2^16 entries, far below a slab
  LDA_TRY(ent.get(std::min<size_t>(size_t(o - at), kSlabEntries)));
  std::vector<uint32_t> rel(rows);
  for (size_t a = 0; a < docs;) {
    size_t b = a, total = 0;
    for (; b < docs && b - a < rows && total + n[b] <= kSlabEntries; ++b) {
      rel[b - a] = uint32_t(total);
      total += n[b];
    }
    LDA_TRY(num.put(rel.data(), b - a));
    HIP_TRY(h, launch_export_d(d, int64_t(a), int64_t(b - a), num.ptr, ent.ptr, h->stream));
    int32_t *tp = topic + off[a], *ct = count + off[a];
    LDA_TRY(read_back(h, crew, ent, total, [tp, ct](const uint32_t *src, size_t first, size_t m) {
      for (size_t i = 0; i < m; ++i) {
        tp[first + i] = int32_t(src[i] >> 16);
        ct[first + i] = int32_t(src[i] & 0xFFFFu);
      }
    }));
    HIP_TRY(h, hipStreamSynchronize(h->stream));  // rel is rewritten
    a = b;
  }
  return LDA_OK;
}

lda_status export_w(lda_handle *h, Crew &crew, const DevState &d, const Params &p, int64_t *off, int32_t *topic,
                    int32_t *count) {
  const Layout &L = h->L;
  const size_t np = size_t(p.n_present), V = size_t(L.V), rows = std::min(V, kSlabRows);
  Scratch<uint32_t> num(h), row(h);
  Scratch<uint2> ent(h);
  LDA_TRY(num.get(std::max(np, rows)));
  HIP_TRY(h, launch_word_nnz(d, p, num.ptr, h->stream));
  std::vector<uint32_t> n(np);
  LDA_TRY(read_back(h, crew, num, np, [&](const uint32_t *src, size_t first, size_t k) {
    std::memcpy(n.data() + first, src, k * sizeof(uint32_t));
  }));
  auto words = [&](size_t v) { return size_t(L.relabel[v]) < np ? size_t(n[size_t(L.relabel[v])]) : size_t(0); };
  int64_t o = 0;
  for (size_t v = 0; v < V; ++v) {
    off[v] = o;
    o += int64_t(words(v));
  }
  off[V] = o;
  // a row has at most K <= 32,768 entries, far below a slab
  LDA_TRY(ent.get(std::min<size_t>(size_t(o), kSlabEntries)));
  LDA_TRY(row.get(rows));
  std::vector<uint32_t> rel(rows), ids(rows);
  for (size_t a = 0; a < V;) {
    size_t b = a, total = 0, m = 0;
    for (; b < V && m < rows && total + words(b) <= kSlabEntries; ++b) {
      if (!words(b)) continue;
      rel[m] = uint32_t(total);
      ids[m++] = uint32_t(L.relabel[b]);
      total += words(b);
    }
    if (m) {
      LDA_TRY(num.put(rel.data(), m));
      LDA_TRY(row.put(ids.data(), m));
      HIP_TRY(h, launch_export_w(d, p, row.ptr, num.ptr, int64_t(m), ent.ptr, h->stream));
      int32_t *tp = topic + off[a], *ct = count + off[a];
      LDA_TRY(read_back(h, crew, ent, total, [tp, ct](const uint2 *src, size_t first, size_t k) {
        for (size_t i = 0; i < k; ++i) {
          tp[first + i] = int32_t(src[i].x);
          ct[first + i] = int32_t(src[i].y);
        }
      }));
      HIP_TRY(h, hipStreamSynchronize(h->stream));  // rel and ids are rewritten
    }
    a = b;
  }
  return LDA_OK;
}

}  // namespace lda
