// Page bookkeeping of paged storage on the host: which pages a sequence's table names, how many tables name a page,
// and the pages nobody uses.  Plain loops over small arrays of the caller's; no device is touched.
//
// A beam search does this between every two steps, so its time adds to every token: at 132 sequences the same
// bookkeeping in the Python session took 0.75 ms a token against 28 us of kernels; here it takes a few microseconds.
#include "../../include/mtla.h"

namespace {

// Highest page (index into a table row) that `len` tokens reach, plus one.
inline int pages_of(const mtla_page_book* k, int64_t len) {
  const int64_t slots = (len + k->stride - 1) / k->stride;
  const int64_t n = (slots + k->page_slots - 1) / k->page_slots;
  return (int)(n < k->max_pages ? n : k->max_pages);
}

inline int32_t take(mtla_page_book* k) {
  const int32_t p = k->free_ring[k->free_head];
  if (++k->free_head == k->n_pages) k->free_head = 0;
  --k->free_count;
  k->refs[p] = 1;
  return p;
}

inline void give(mtla_page_book* k, int32_t p) {
  if (--k->refs[p] != 0) return;
  int64_t at = k->free_head + k->free_count;
  if (at >= k->n_pages) at -= k->n_pages;
  k->free_ring[at] = p;
  ++k->free_count;
}

inline bool valid(const mtla_page_book* k) {
  return k && k->table && k->len && k->next_table && k->next_len && k->refs && k->free_ring && k->max_batch > 0 &&
         k->max_pages > 0 && k->n_pages > 0 && k->page_slots > 0 && k->stride > 0 && k->max_slots > 0;
}

}  // namespace

extern "C" {

int32_t mtla_pages_reserve(mtla_page_book* k, const int32_t* n_new, int32_t batch) {
  if (!valid(k) || batch < 1 || batch > k->max_batch) return -1;
  // the entries of a row are filled from the front, so what is missing lies behind the last one filled
  int64_t missing = 0;
  for (int b = 0; b < batch; ++b) {
    const int32_t* row = k->table + (int64_t)b * k->max_pages;
    for (int e = pages_of(k, k->len[b] + (n_new ? n_new[b] : 1)) - 1; e >= 0 && row[e] < 0; --e) ++missing;
  }
  if (missing == 0) return 0;
  if (missing > k->free_count) return -2;
  for (int b = 0; b < batch; ++b) {
    int32_t* row = k->table + (int64_t)b * k->max_pages;
    const int need = pages_of(k, k->len[b] + (n_new ? n_new[b] : 1));
    int first = need;
    while (first > 0 && row[first - 1] < 0) --first;
    for (int e = first; e < need; ++e) row[e] = take(k);
  }
  return (int32_t)(missing < 0x7fffffff ? missing : 0x7fffffff);
}

int32_t mtla_pages_fork(mtla_page_book* k, const int32_t* src_index, int32_t batch, int32_t* fresh_pages) {
  if (!valid(k) || !src_index || !fresh_pages || batch < 1 || batch > k->max_batch) return -1;
  const int64_t row_len = k->max_pages;
  // how often a source is continued (counted in next_len, which is rewritten below)
  for (int b = 0; b < k->max_batch; ++b) k->next_len[b] = 0;
  for (int b = 0; b < batch; ++b) {
    if (src_index[b] < 0 || src_index[b] >= k->max_batch) return -1;
    ++k->next_len[src_index[b]];
  }
  // the page a source's next token goes to: the continuation's own, taken over from a source with one continuation
  auto write_page = [&](int s) {
    int64_t next = k->len[s] / k->stride;
    if (next > k->max_slots - 1) next = k->max_slots - 1;
    return (int)(next / k->page_slots);
  };
  int64_t wanted = 0;
  for (int b = 0; b < batch; ++b) {
    const int s = src_index[b];
    fresh_pages[b] = k->next_len[s] == 1 ? k->table[s * row_len + write_page(s)] : -1;
    if (fresh_pages[b] < 0) ++wanted;
  }
  if (wanted > k->free_count) return -2;
  for (int b = 0; b < k->max_batch; ++b) {
    int32_t* row = k->next_table + b * row_len;
    int n = 0;
    k->next_len[b] = 0;
    if (b < batch) {
      const int s = src_index[b], pw = write_page(s);
      const int32_t* from = k->table + s * row_len;
      for (; n < pw; ++n) {
        row[n] = from[n];
        if (row[n] >= 0) ++k->refs[row[n]];
      }
      if (fresh_pages[b] >= 0) ++k->refs[fresh_pages[b]];
      else fresh_pages[b] = take(k);
      row[n++] = fresh_pages[b];
      k->next_len[b] = k->len[s];
    }
    for (; n < row_len; ++n) row[n] = -1;
  }
  for (int64_t e = 0; e < k->max_batch * row_len; ++e)  // the old sequences let go of their pages
    if (k->table[e] >= 0) give(k, k->table[e]);
  int32_t* t = k->table;
  k->table = k->next_table;
  k->next_table = t;
  int64_t* l = k->len;
  k->len = k->next_len;
  k->next_len = l;
  return 0;
}

}  // extern "C"
