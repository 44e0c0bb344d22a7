"""How an open cuts a file into passes and the long streams of a pass into groups
(pq_open_passes.hpp, compiled for the CPU): every page and stream once and in order,
the decompressed bytes, chain tables and segments of each within their caps unless
it is one page or one stream, and no cut that is not needed.  Uncompressed files too:
their pages have no decompressed bytes, so only the tables bound a pass."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

MAIN = r"""
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include "pq_open_passes.hpp"
using namespace pqk;
#define NEED(x) do { if (!(x)) { printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)

struct File { uint32_t pages, rows, bytes; int enc, type; bool optional, compressed; };

static int passes(const File& F, size_t want) {
  std::vector<uint64_t> scr(F.pages + 1, 0), tab(F.pages + 1, 0);
  for (uint32_t p = 0; p < F.pages; ++p) {
    PageDev pg;
    memset(&pg, 0, sizeof(pg));
    pg.kind = PAGE_DATA;
    pg.encoding = (uint8_t)F.enc;
    pg.num_values = (int32_t)F.rows;
    pg.uncomp_size = F.bytes;
    scr[p + 1] = scr[p] + (F.compressed ? F.bytes + 16 : 0);
    const uint64_t b = chain_table_bytes(pg, F.type, F.optional);
    // what the pass allocates for the page: level pieces, index pieces or DELTA blocks, its list entries
    uint64_t need = sizeof(IxPage) + 8;
    if (F.optional) need += 9ull * chain_pieces(F.rows / 8 + F.rows / 504 + 8);
    if (F.enc == E_RLE_DICT) need += 5ull * chain_pieces(F.bytes);
    if (F.enc == E_DELTA) need += 4 * ((F.rows + 127ull) / 128 + 1);
    NEED(b >= need);
    tab[p + 1] = tab[p] + b;
  }
  const std::vector<uint32_t> at = cut_passes(scr, tab, F.pages);
  NEED(at.front() == 0 && at.back() == F.pages);
  for (size_t k = 0; k + 1 < at.size(); ++k) {
    NEED(at[k] < at[k + 1]);
    auto over = [&](uint32_t a, uint32_t b) {
      return scr[b] - scr[a] > OPEN_SCRATCH_CAP || tab[b] - tab[a] > OPEN_TABLE_CAP;
    };
    NEED(!over(at[k], at[k + 1]) || at[k + 1] == at[k] + 1);
    if (k + 2 < at.size()) NEED(over(at[k], at[k + 1] + 1));
  }
  if (want) NEED(at.size() - 1 == want);
  else NEED(at.size() - 1 > 3);
  return 0;
}

static int groups(const std::vector<uint32_t>& lens) {
  std::vector<std::pair<uint32_t, uint32_t>> l;
  for (uint32_t i = 0; i < lens.size(); ++i) l.push_back({lens[i], i});
  const std::vector<uint32_t> at = cut_groups(l, (uint32_t)l.size());
  NEED(at.back() == l.size() && (at.front() == 0 || l.empty()));
  for (size_t k = 0; k + 1 < at.size(); ++k) {
    NEED(at[k] < at[k + 1]);
    uint64_t n = 0;
    for (uint32_t i = at[k]; i < at[k + 1]; ++i) n += stream_segs(l[i].first);
    NEED(n <= OPEN_SEGS || at[k + 1] == at[k] + 1);
    if (k + 2 < at.size()) NEED(n + stream_segs(l[at[k + 1]].first) > OPEN_SEGS);
  }
  return 0;
}

int main() {
  const uint32_t M = 1 << 20;
  int bad = 0;
  bad |= passes({1, 1, 1, E_PLAIN, T_INT32, false, false}, 1);
  bad |= passes({15000, 524288, M, E_RLE_DICT, T_INT32, true, false}, 0);     // 15 GB of 16-bit indices, uncompressed
  bad |= passes({1000, 524288, M, E_RLE_DICT, T_INT32, true, false}, 1);      // 1 GB of them
  bad |= passes({15000, 131072, M, E_PLAIN, T_INT64, true, false}, 1);        // PLAIN: levels alone
  bad |= passes({60000, 524288, 4096, E_DELTA, T_INT64, false, false}, 0);     // constant deltas: blocks of a few bytes
  bad |= passes({5, 524288, 1u << 30, E_PLAIN, T_INT64, true, true}, 5);      // pages above the window
  bad |= passes({4000, 524288, M, E_PLAIN, T_INT64, true, true}, 0);
  bad |= passes({4, 1u << 30, 2000u * M, E_RLE_DICT, T_INT32, true, false}, 4);
  bad |= groups({});
  bad |= groups({2000u * M, 2000u * M, 100, 100});
  bad |= groups(std::vector<uint32_t>(300, 8u * M));
  bad |= groups(std::vector<uint32_t>(9000, 32768 - 15));
  bad |= groups(std::vector<uint32_t>(9000, 32768 - 14));
  if (!bad) printf("ok\n");
  return bad;
}
"""


def test_passes_and_groups(tmp_path):
    src, exe = tmp_path / "main.cpp", tmp_path / "main"
    src.write_text(MAIN)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-D__host__=", "-D__device__=",
                           "-I", os.path.join(ROOT, "paper_2602_17335_amd", "csrc"), str(src), "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout
