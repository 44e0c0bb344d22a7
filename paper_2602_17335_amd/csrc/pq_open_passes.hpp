// pq_open_passes.hpp -- how an open cuts a file's pages into passes and the
// segments of a pass's long streams into groups, so that its temporary device memory
// is bounded (host only).
#pragma once
#include <stdint.h>

#include <algorithm>
#include <utility>
#include <vector>

#include "pq_internal.h"

namespace pqk {

// Decompressed bytes of the data pages indexed together.
constexpr uint64_t OPEN_SCRATCH_CAP = 512ull << 20;
// Bytes of their chain tables.  (Each pass costs a few round trips; the tables of
// the 64M-row uncompressed wide table, 15 GB, take 0.2 GiB.)
constexpr uint64_t OPEN_TABLE_CAP = 256ull << 20;
// Segments whose exits are held at once, 13 KiB each (52 MiB; 128 MiB of streams).
constexpr uint32_t OPEN_SEGS = 4096;

// Bytes of the chain tables of a data page, from its header: 9 per piece of 32 level
// bytes, 5 per piece of dictionary indices, 4 per 128 DELTA values, its entry in
// the page list.  The level bytes of a V1 page are taken as those of runs of eight
// rows or more.
inline uint64_t chain_table_bytes(const PageDev& pg, int32_t type, bool optional) {
  uint64_t n = sizeof(IxPage) + 12;
  const uint64_t nv = pg.num_values > 0 ? (uint64_t)pg.num_values : 0, body = pg.uncomp_size;
  if (optional && nv) {
    const uint64_t lv = pg.kind == PAGE_DATA_V2 ? (uint64_t)(pg.def_len > 0 ? pg.def_len : 0) : std::min(body, nv / 4 + 64);
    n += 9ull * chain_pieces(lv);
  }
  if (pg.encoding == E_PLAIN_DICT || pg.encoding == E_RLE_DICT) n += 5ull * chain_pieces(body);
  else if (pg.encoding == E_DELTA || (pg.encoding == E_DLBA && type == T_BYTE_ARRAY)) n += 4 * (nv / 128 + 2);
  return n;
}

// The first pages of the passes over n pages (and n): runs of pages, each as long as
// the differences of both prefixes (n + 1 entries) stay within the caps, one page at
// least.
inline std::vector<uint32_t> cut_passes(const std::vector<uint64_t>& scratch, const std::vector<uint64_t>& tables, uint32_t n) {
  std::vector<uint32_t> at;
  for (uint32_t p = 0; p < n;) {
    at.push_back(p);
    uint32_t p1 = p + 1;
    while (p1 < n && scratch[p1 + 1] - scratch[p] <= OPEN_SCRATCH_CAP && tables[p1 + 1] - tables[p] <= OPEN_TABLE_CAP) ++p1;
    p = p1;
  }
  at.push_back(n);
  return at;
}

// 32 KiB segments of a stream of len bytes from any byte of its first 16.
inline uint32_t stream_segs(uint32_t len) { return (uint32_t)(((uint64_t)len + 15 + 32767) / 32768); }

// The streams l[0, n) (bytes, page) in runs of at most OPEN_SEGS segments, one stream
// at least: the first stream of each, and n.
inline std::vector<uint32_t> cut_groups(const std::vector<std::pair<uint32_t, uint32_t>>& l, uint32_t n) {
  std::vector<uint32_t> at;
  for (uint32_t i = 0; i < n;) {
    at.push_back(i);
    uint64_t segs = stream_segs(l[i].first);
    uint32_t j = i + 1;
    while (j < n && segs + stream_segs(l[j].first) <= OPEN_SEGS) segs += stream_segs(l[j++].first);
    i = j;
  }
  at.push_back(n);
  return at;
}

}  // namespace pqk
