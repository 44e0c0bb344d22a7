// pq_open_kernels.hip -- kernels that run once when a file is opened:
//   k_walk   page-header walk of every column chunk -> device page table
//   k_layout  stream layout of every page
//   k_levels, k_strings, k_di, k_dl  the element chains of level streams, string
//            lengths, dictionary-index runs and DELTA blocks (pq_chain.hpp)
//   k_seg_cand, k_seg_link, k_seg_fill, k_seg_base, k_str_ck, k_dl_ck  the same for
//            the segments of long value streams side by side
//   k_tiles, k_values, k_value_tiles  tile entries and checkpoints from them
//   k_index  the whole index of one page by one wave, for pages whose
//            chains the kernels above leave (and to say what is wrong with
//            malformed ones)
#include <hip/hip_runtime.h>

#include "pq_chain.hpp"
#include "pq_device.hpp"
#include "pq_internal.h"

namespace pqk {

// Hybrid-run cursor used by the index kernels (one lane).
struct RunCur {
  uint64_t hp;     // header position of the current run
  uint64_t next;   // position after the current run
  int64_t start;   // first value index of the current run
  uint64_t n;      // values in the run
  int bp;          // bit-packed?
  uint64_t pay;    // payload byte position (bit-packed)
  uint32_t val;    // RLE value
};

// Stream reader of one wave for k_index: all 64 lanes walk the same stream
// in lockstep (the walk is sequential; every lane computes the same values),
// served from a WIN-byte LDS window that the wave refills with coalesced
// 16-byte loads (one memory round trip per window instead of one per 16
// bytes); every read is an LDS read (all lanes read the same address, a
// broadcast).  The window keeps
// 256 bytes before the position that moved it, for the short look-backs of
// the walk (a run's payload).  Bytes at or past `lim` read as zero.
constexpr uint32_t WIN = 4096;
static_assert(NLCK == 64, "lane k of a wave writes level checkpoint k of a tile");
typedef uint32_t wr_u4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) wr_u4 lds_u4;

// Refills the window for position a (a multiple of 16); returns its start.
__device__ __noinline__ uint64_t wr_refill(const uint8_t* base, uint64_t lim, lds_u4* win, uint64_t a) {
  uint64_t wpos = a > 256 ? a - 256 : 0;
  wpos = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(wpos >> 32)) << 32) |
         (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)wpos);
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  const uint32_t lane = threadIdx.x & 63;
#pragma unroll
  for (uint32_t j = 0; j < WIN / 16 / 64; ++j) {
    const uint32_t k = lane + 64 * j;
    const uint64_t g = wpos + 16ull * k;
    wr_u4 v = {0u, 0u, 0u, 0u};
    if (g + 16 <= lim) v = *reinterpret_cast<const wr_u4*>(base + g);
    win[k] = v;
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  return wpos;
}

struct WR {
  const uint8_t* base;
  uint64_t lim;   // bytes of base that may be read (a multiple of 16)
  uint64_t wpos;  // window start (a multiple of 16)
  lds_u4* win;
  __device__ __forceinline__ void init(const uint8_t* b, uint64_t l, lds_u4* w) {
    base = b;
    lim = l;
    win = w;
    wpos = ~0ull;
  }
  // the window holds bytes [off, off + n)
  __device__ __forceinline__ void ensure(uint64_t off, uint32_t n) {
    if (off < wpos || off + n - wpos > WIN) wpos = wr_refill(base, lim, win, off & ~15ull);
  }
  // every lane reads the same byte, so the value is moved to a scalar
  // register: the walk that follows runs on the scalar unit, with scalar
  // branches instead of exec-mask updates
  __device__ __forceinline__ uint32_t byte(uint64_t off) {
    ensure(off, 1);
    return (uint32_t)__builtin_amdgcn_readfirstlane(
        (int)reinterpret_cast<__attribute__((address_space(3))) uint8_t*>(win)[off - wpos]);
  }
  __device__ __forceinline__ uint32_t u32(uint64_t off) {
    ensure(off, 8);  // both aligned dwords holding bytes [off, off + 4)
    const uint32_t o = (uint32_t)(off - wpos);
    const __attribute__((address_space(3))) uint32_t* w32 = reinterpret_cast<__attribute__((address_space(3))) uint32_t*>(win);
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)__builtin_amdgcn_alignbyte(w32[(o >> 2) + 1], w32[o >> 2], o & 3));
  }
};

// Wave reader with the window in registers: 256 bytes, four per lane; a
// read at a wave-uniform offset is one v_readlane, so a walk whose every
// position is wave-uniform waits on memory once per window, not per byte.
// Every lane must take part in every read.  It reads a global buffer
// readable up to lim (a multiple of 16); bytes at or past lim read as zero.
struct GRegWin {
  const uint8_t* base;
  uint64_t lim, wl;  // window start (a multiple of 4)
  uint32_t v;
  __device__ __forceinline__ void init(const uint8_t* b, uint64_t l) {
    base = b;
    lim = l;
    wl = 1ull << 63;  // far from every offset: the first read fills the window
    v = 0;
  }
  __device__ __forceinline__ uint32_t byte(uint64_t off) {
    if (off - wl >= 256) {
      wl = off & ~3ull;
      const uint64_t a = wl + 4ull * (threadIdx.x & 63);
      v = a + 4 <= lim ? *reinterpret_cast<const uint32_t*>(base + a) : 0u;
    }
    const uint32_t o = (uint32_t)(off - wl);
    return ((uint32_t)__builtin_amdgcn_readlane((int)v, (int)(o >> 2)) >> (8 * (o & 3))) & 0xffu;
  }
};

// The page table entry of a page whose header h was parsed, payload first.
__device__ __forceinline__ PageDev make_page(const PageHdr& h, uint64_t payload, uint32_t chunk) {
  PageDev p;
  p.payload = payload;
  p.comp_size = (uint32_t)h.comp;
  p.uncomp_size = (uint32_t)h.unc;
  p.num_values = h.nv;
  p.num_nulls = h.type == PAGE_DATA_V2 ? h.nnulls : -1;
  p.chunk = chunk;
  p.kind = (uint8_t)h.type;
  p.encoding = (uint8_t)h.enc;
  p.v2_compressed = (uint8_t)(h.type == PAGE_DATA_V2 ? h.is_comp : 1);
  p.flags = 0;
  p.def_len = h.type == PAGE_DATA_V2 ? h.def_len : 0;
  p.sbit0 = 0;  // (and no repetition levels: such pages are refused)
  p.def_off = 0; p.val_off = 0; p.val_len = 0;
  p.scratch_len = 0; p.scratch_off = 0; p.row0 = 0;
  p.tile_begin = 0; p.nonnull = 0; p.strck_begin = 0; p.dict_page = ~0u; p.dict_maxlen = 0;
  p.enc_w = 0; p.enc_m = 0; p.delta_first = 0; p.blocks_at = 0; p.sblk_begin = 0; p.chars_at = 0;
  return p;
}

// One wave per column chunk.  Walks PageHeader, payload, PageHeader, ...
// from the chunk start until the chunk's byte range is consumed, checking
// every header.  With `pages == nullptr` it counts pages (first pass) and,
// when `rec` is given, records the header offsets of the first rec_cap[chunk]
// pages at rec[rec_base[chunk] ..] (setting *overflow past that); otherwise
// it writes the page table entries at page_base[chunk].  Each header is
// read through a register window that the wave fills with one coalesced
// load (the headers of a chunk lie a page apart, so a byte-serial reader
// would wait on memory for every 16 bytes); every lane parses, lane 0
// stores.
__global__ __launch_bounds__(64) void k_walk(const uint8_t* file, uint64_t file_lim, const ChunkDev* chunks,
                                             int nchunks, uint32_t* counts, const uint32_t* page_base,
                                             PageDev* pages, uint32_t* err, uint64_t* rec, const uint32_t* rec_base,
                                             const uint32_t* rec_cap, uint32_t* overflow) {
  const int q = blockIdx.x;
  if (q >= nchunks) return;
  const bool lead = threadIdx.x == 0;
  ChunkDev c = chunks[q];
  GRegWin r;
  r.init(file, file_lim);
  uint64_t pos = c.start;
  uint32_t n = 0;
  int64_t rows = 0;
  bool seen_data = false, seen_dict = false;
  const uint32_t cap = rec ? rec_cap[q] : 0u;
  while (pos < c.end) {
    PageHdr h;
    const uint64_t hpos = pos;
    if (!parse_page_header(r, pos, c.end, h) || h.type < 0 || h.unc < 0 || h.comp < 0) { if (lead) set_err(err, ERR_HEADER, q); return; }
    uint64_t payload = pos;
    if ((uint64_t)h.comp > c.end - payload) { if (lead) set_err(err, ERR_CHUNK_BOUNDS, q); return; }
    pos = payload + (uint64_t)h.comp;
    if (h.type == PAGE_DICT) {
      if (seen_data || seen_dict) { if (lead) set_err(err, ERR_PAGE_ORDER, q); return; }
      if (!h.has_sub || h.nv < 0) { if (lead) set_err(err, ERR_HEADER, q); return; }
      if (h.enc != E_PLAIN && h.enc != E_PLAIN_DICT) { if (lead) set_err(err, ERR_UNSUPPORTED, q); return; }
      if (c.codec == 0 && h.comp != h.unc) { if (lead) set_err(err, ERR_HEADER, q); return; }
      seen_dict = true;
    } else if (h.type == PAGE_DATA || h.type == PAGE_DATA_V2) {
      if (!h.has_sub || h.nv < 0) { if (lead) set_err(err, ERR_HEADER, q); return; }
      bool enc_ok = h.enc == E_PLAIN || h.enc == E_PLAIN_DICT || h.enc == E_RLE_DICT ||
                    (h.enc == E_DELTA && (c.type == T_INT32 || c.type == T_INT64)) ||
                    (h.enc == E_BSS && c.type != T_BYTE_ARRAY) ||
                    ((h.enc == E_DLBA || h.enc == E_DBA) && c.type == T_BYTE_ARRAY);
      // (DELTA_BYTE_ARRAY pages open, and are reported as unsupported only
      // when a scan selects their column)
      if (!enc_ok) { if (lead) set_err(err, ERR_UNSUPPORTED, q); return; }
      if (h.type == PAGE_DATA_V2) {
        if (h.rep_len != 0) { if (lead) set_err(err, ERR_UNSUPPORTED, q); return; }
        if (h.def_len < 0 || h.nrows != h.nv || h.def_len > h.comp || h.def_len > h.unc || h.nnulls < 0 ||
            (!c.optional && (h.def_len != 0 || h.nnulls != 0))) { if (lead) set_err(err, ERR_V2, q); return; }
        bool compressed = c.codec == 1 && h.is_comp;
        if (!compressed && h.comp != h.unc) { if (lead) set_err(err, ERR_V2, q); return; }
      } else if (c.codec == 0 && h.comp != h.unc) { if (lead) set_err(err, ERR_HEADER, q); return; }
      rows += h.nv;
      if (rows > c.rows) { if (lead) set_err(err, ERR_ROWS, q); return; }
      seen_data = true;
    } else {
      continue;  // index pages and unknown page types are skipped
    }
    if (pages) {
      const PageDev p = make_page(h, payload, (uint32_t)q);
      if (lead) pages[page_base[q] + n] = p;
    } else if (rec && lead) {
      if (n < cap) rec[rec_base[q] + n] = hpos;
      else *overflow = 1;
    }
    ++n;
  }
  if (pos != c.end || rows != c.rows) { if (lead) set_err(err, ERR_ROWS, q); return; }
  if (counts && lead) counts[q] = n;
}

// One lane per page recorded by k_walk's first pass: parses its header again
// (already checked there) into the page table.  page_chunk[i] is page i's
// chunk; its header offset is rec[rec_base[chunk] + i - page_base[chunk]].
__global__ void k_walk_rec(const uint8_t* file, const ChunkDev* chunks, const uint64_t* rec, const uint32_t* rec_base,
                           const uint32_t* page_base, const uint32_t* page_chunk, uint32_t npages, PageDev* pages,
                           uint32_t* err) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= npages) return;
  const uint32_t q = page_chunk[i];
  const uint64_t end = chunks[q].end;
  uint64_t pos = rec[rec_base[q] + (i - page_base[q])];
  BR r;
  r.init(file);
  PageHdr h;
  if (!parse_page_header(r, pos, end, h)) { set_err(err, ERR_HEADER, q); return; }
  pages[i] = make_page(h, pos, q);
}

// Reads the run header at cur.next; returns false when the stream ends or a
// run leaves it.
__device__ inline bool run_next(WR& r, uint64_t end, uint32_t w, RunCur& c) {
  uint64_t pos = c.next;
  c.start += (int64_t)c.n;
  c.hp = pos;
  bool bad = false;
  uint64_t h = br_uleb(r, pos, end, bad);
  if (bad) return false;
  if (h & 1) {
    uint64_t g = h >> 1;
    if (g > (1ull << 28)) return false;
    c.bp = 1;
    c.n = g * 8;
    c.pay = pos;
    uint64_t nb = g * w;
    if (nb > end - pos) return false;
    c.next = pos + nb;
    c.val = 0;
  } else {
    c.bp = 0;
    c.n = h >> 1;
    uint32_t vb = (w + 7) / 8;
    if (vb > end - pos) return false;
    uint32_t v = 0;
    for (uint32_t j = 0; j < vb; ++j) v |= r.byte(pos + j) << (8 * j);
    c.val = v;
    c.pay = pos;
    c.next = pos + vb;
  }
  return true;
}

// number of set bits among the first `k` values of a bit-packed w=1 run
// (1024 bits per window check, then a dword per 32 bits straight from LDS)
__device__ inline uint32_t bp_popcount(WR& r, uint64_t pay, uint64_t k) {
  uint32_t s = 0;
  const __attribute__((address_space(3))) uint32_t* w32 =
      reinterpret_cast<const __attribute__((address_space(3))) uint32_t*>(r.win);
  for (uint64_t b0 = 0; b0 < k; b0 += 1024) {
    const uint32_t kk = (uint32_t)min(k - b0, (uint64_t)1024);
    const uint64_t off = pay + (b0 >> 3);
    r.ensure(off, 136);  // the 128 bytes and the dword after them
    const uint32_t o = (uint32_t)(off - r.wpos), sh = o & 3, d = o >> 2;
    for (uint32_t i = 0; 32 * i < kk; ++i) {
      uint32_t v = __builtin_amdgcn_alignbyte(w32[d + i + 1], w32[d + i], sh);
      const uint32_t left = kk - 32 * i;
      if (left < 32) v &= (1u << left) - 1u;
      s += __popc(v);
    }
  }
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)s);
}

// Checkpoint of value `target` inside run c of a w-bit hybrid stream whose
// tile entry sits at absolute position `entry`.
__device__ __forceinline__ Ck make_ck(const RunCur& c, int64_t target, uint32_t w, uint64_t entry) {
  Ck k;
  k.at = CK_NONE;
  k.info = 0;
  const uint64_t skip = (uint64_t)(target - c.start);
  const uint64_t left = min(c.n - skip, (uint64_t)CK_LEFT);
  if (c.bp) {
    const uint64_t bit = c.pay * 8 + skip * w;
    const uint64_t off = (bit >> 3) - entry;
    if (off >= CK_NONE) return k;
    k.at = (uint32_t)off;
    k.info = 0x80000000u | ((uint32_t)(bit & 7) << 28) | (uint32_t)left;
  } else {
    const uint64_t off = c.hp - entry;
    if (off >= CK_NONE) return k;
    k.at = (uint32_t)off;
    k.info = (uint32_t)left;
  }
  return k;
}

// Level checkpoint (format in pq_internal.h) of row `target` inside run c of
// a level stream whose tile entry sits at absolute position `entry`.
__device__ __forceinline__ uint32_t make_lck(const RunCur& c, int64_t target, uint64_t entry) {
  const uint64_t skip = (uint64_t)(target - c.start);
  const uint64_t left = min(c.n - skip, (uint64_t)LROWS);
  uint64_t off;
  uint32_t x;
  if (c.bp) {
    const uint64_t bit = c.pay * 8 + skip;
    off = (bit >> 3) - entry;
    x = (1u << 19) | ((uint32_t)(bit & 7) << 16);
  } else {
    off = c.next - entry;
    x = (c.val & 1u) << 20;
  }
  if (off > 0xffffu) return LCK_NONE;
  return (uint32_t)off | x | ((uint32_t)left << 21);
}

__device__ __forceinline__ Ck ck_at(uint64_t off) {
  Ck k;
  k.at = off < CK_NONE ? (uint32_t)off : CK_NONE;
  k.info = 0;
  return k;
}

__device__ __forceinline__ Ck ck_none() {
  Ck k;
  k.at = CK_NONE;
  k.info = 0;
  return k;
}

// The pages whose flag is set, one wave each (a 64-thread workgroup; every
// lane runs the same walk and stores the same values).  `scratch` holds every
// compressed page decompressed at its file-wide scratch offset; file_lim and
// scratch_lim are the readable bytes of the two buffers (multiples of 16).
__global__ __launch_bounds__(64) void k_index(const uint8_t* file, const uint8_t* scratch, PageDev* pages,
                                              const IxPage* ixs, const uint32_t* flag, const ChunkDev* chunks,
                                              TileDev* tiles, uint32_t* strck, uint32_t* ckl, Ck* ckv, uint32_t* err,
                                              uint64_t file_lim, uint64_t scratch_lim, const uint8_t* xscratch,
                                              uint64_t xscratch_lim, const PageX* pagex) {
  __shared__ wr_u4 s_win[WIN / 16];
  // DELTA pages of at most TC tiles: first value, value count and value
  // entry of every tile, so that the block walk reads no tile from memory
  constexpr uint32_t TC = 2048;
  __shared__ uint32_t s_k0[TC], s_nn[TC], s_vp[TC];
  if (!flag[blockIdx.x] || *(volatile uint32_t*)err != 0) return;
  const int p = (int)ixs[blockIdx.x].page;
  PageDev pg = pages[p];
  ChunkDev ch = chunks[pg.chunk];
  const bool in_scratch = pg.scratch_len > 0;
  WR r;
  lds_u4* win = (lds_u4*)&s_win[0];
  // Stores that nothing in this kernel reads back (checkpoints) come from
  // lane 0 alone.
  // Tiles and the page entry are stored by every lane (each lane reads back
  // its own stores).
  const bool lead = (threadIdx.x & 63) == 0;
  auto lim_of = [&](const uint8_t* b) { return b == file ? file_lim : (b == xscratch ? xscratch_lim : scratch_lim); };

  if (pg.kind == PAGE_DICT) {
    const uint8_t* base = in_scratch ? scratch : file;
    uint64_t off = in_scratch ? pg.scratch_off : pg.payload;
    uint64_t blen = pg.uncomp_size;
    pg.val_off = off;
    pg.val_len = (uint32_t)blen;
    pg.flags = in_scratch ? 2 : 0;
    if (ch.type == T_BYTE_ARRAY) {
      // the length-prefix chain in 32-bit positions (a page is below 4 GiB):
      // q in the page body, o in the LDS window, one LDS read per entry; the
      // window moves when an entry's length prefix would leave it.  Every
      // lane reads the same length, which is moved to a scalar register, so
      // the chain and its checks run on the scalar unit
      const uint64_t blim = lim_of(base);
      const uint32_t n = pg.num_values > 0 ? (uint32_t)pg.num_values : 0u;
      const uint32_t bl = (uint32_t)blen;
      const __attribute__((address_space(3))) uint32_t* w32 =
          reinterpret_cast<const __attribute__((address_space(3))) uint32_t*>(win);
      uint32_t q = 0, maxlen = 0, k = 0;
      while (k < n) {
        const uint64_t wpos = wr_refill(base, blim, win, (off + q) & ~15ull);
        uint32_t o = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(off + q - wpos));  // below 272
        while (k < n && o + 8 <= WIN) {
          if ((k % STR_CK) == 0 && lead) strck[pg.strck_begin + k / STR_CK] = q;
          if (bl - q < 4) { set_err(err, ERR_STRING, p); return; }
          const uint32_t l = (uint32_t)__builtin_amdgcn_readfirstlane(
              (int)__builtin_amdgcn_alignbyte(w32[(o >> 2) + 1], w32[o >> 2], o & 3));
          if (l > bl - q - 4) { set_err(err, ERR_STRING, p); return; }
          q += 4 + l;
          o = l < WIN ? o + 4 + l : WIN;
          maxlen = max(maxlen, l);
          ++k;
        }
      }
      pg.dict_maxlen = maxlen;
    } else {
      uint64_t w = ch.type == T_INT32 ? 4 : 8;
      if ((uint64_t)pg.num_values * w > blen) { set_err(err, ERR_VALUES, p); return; }
    }
    pages[p] = pg;
    return;
  }

  // ---- stream layout of a data page (as k_layout found it) ----
  const uint8_t* dbase = (pg.flags & 1) ? scratch : file;
  const uint8_t* vbase = (pg.flags & 4) ? xscratch : ((pg.flags & 2) ? scratch : file);
  const uint64_t def_off = pg.def_off, def_len = (uint64_t)pg.def_len, val_off = pg.val_off, val_len = pg.val_len;

  const int64_t nv = pg.num_values;
  const uint32_t ntiles = (uint32_t)((nv + TILE_ROWS - 1) / TILE_ROWS);

  // ---- definition levels: tile entry points, sub-tile checkpoints, non-null counts ----
  uint32_t nonnull = 0;
  if (ch.optional) {
    r.init(dbase, lim_of(dbase), win);
    const uint64_t end = def_off + def_len;
    RunCur c;
    c.next = def_off; c.start = 0; c.n = 0; c.bp = 0; c.val = 0; c.pay = 0; c.hp = def_off;
    uint64_t before = 0;  // valid rows in runs before the current one
    bool have = false;
    TileDev td;
    for (int64_t target = 0; target < nv; target += LROWS) {
      while (!have || c.start + (int64_t)c.n <= target) {
        if (have) before += c.bp ? bp_popcount(r, c.pay, c.n) : (uint64_t)c.val * c.n;
        if (!run_next(r, end, 1, c) || (!c.bp && c.val > 1)) { set_err(err, ERR_LEVELS, p); return; }
        have = true;
      }
      const uint64_t skip = (uint64_t)(target - c.start);
      const uint32_t t = (uint32_t)(target / TILE_ROWS), sub = (uint32_t)((target % TILE_ROWS) / LROWS);
      if (sub == 0) {
        td.page = (uint32_t)p;
        td.row0 = (uint32_t)target;
        td.k0 = (uint32_t)(before + (c.bp ? bp_popcount(r, c.pay, skip) : (uint64_t)c.val * skip));
        td.nn = 0;
        td.def_pos = (uint32_t)(c.hp - def_off);
        td.def_skip = (uint32_t)skip;
        td.val_pos = 0;
        td.val_skip = 0;
        tiles[pg.tile_begin + t] = td;
      }
      if (lead) ckl[(size_t)(pg.tile_begin + t) * NLCK + sub] = make_lck(c, target, def_off + td.def_pos);
    }
    // the last tile's checkpoints past the page's rows
    if (nv > 0 && lead)
      for (int64_t target = ((nv + LROWS - 1) / LROWS) * LROWS; target % TILE_ROWS != 0; target += LROWS)
        ckl[(size_t)(pg.tile_begin + (uint32_t)(target / TILE_ROWS)) * NLCK + (target % TILE_ROWS) / LROWS] = LCK_NONE;
    if (nv > 0) {
      while (!have || c.start + (int64_t)c.n < nv) {
        if (have) before += c.bp ? bp_popcount(r, c.pay, c.n) : (uint64_t)c.val * c.n;
        if (!run_next(r, end, 1, c) || (!c.bp && c.val > 1)) { set_err(err, ERR_LEVELS, p); return; }
        have = true;
      }
      const uint64_t part = (uint64_t)(nv - c.start);
      nonnull = (uint32_t)(before + (c.bp ? bp_popcount(r, c.pay, part) : (uint64_t)c.val * part));
    }
  } else {
    nonnull = (uint32_t)nv;
    for (uint32_t t = 0; t < ntiles; ++t) {
      TileDev td;
      td.page = (uint32_t)p;
      td.row0 = t * TILE_ROWS;
      td.k0 = t * TILE_ROWS;
      td.nn = 0;
      td.def_pos = 0; td.def_skip = 0; td.val_pos = 0; td.val_skip = 0;
      tiles[pg.tile_begin + t] = td;
      ckl[(size_t)(pg.tile_begin + t) * NLCK + (threadIdx.x & 63)] = LCK_NONE;  // lane k: checkpoint k
    }
  }
  if (lead)
    for (uint32_t t = 0; t < ntiles; ++t)
      for (int k = 0; k < NSUB; ++k) ckv[(size_t)(pg.tile_begin + t) * NSUB + k] = ck_none();
  if (pg.kind == PAGE_DATA_V2 && (int64_t)pg.num_nulls != nv - (int64_t)nonnull) { set_err(err, ERR_V2, p); return; }
  pg.nonnull = nonnull;
  for (uint32_t t = 0; t < ntiles; ++t) {
    uint32_t k0 = tiles[pg.tile_begin + t].k0;
    uint32_t k1 = t + 1 < ntiles ? tiles[pg.tile_begin + t + 1].k0 : nonnull;
    tiles[pg.tile_begin + t].nn = k1 - k0;
  }

  // ---- value stream entry points ----
  r.init(vbase, lim_of(vbase), win);
  const uint64_t vend = val_off + val_len;
  const int enc = pg.encoding;
  if ((enc == E_PLAIN || enc == E_BSS) && ch.type != T_BYTE_ARRAY) {
    uint64_t w = ch.type == T_INT32 ? 4 : 8;
    if ((uint64_t)nonnull * w > val_len) { set_err(err, ERR_VALUES, p); return; }
  } else if (enc == E_PLAIN || enc == E_DBA) {
    if (enc == E_DBA && pagex[p].x_total != nonnull) { set_err(err, ERR_VALUES, p); return; }
    uint64_t q = val_off;
    uint32_t t = 0;
    for (uint32_t k = 0; k <= nonnull; ++k) {
      while (t < ntiles && tiles[pg.tile_begin + t].k0 == k) {
        tiles[pg.tile_begin + t].val_pos = (uint32_t)(q - val_off);
        if (t > 0) tiles[pg.tile_begin + t - 1].val_skip = (uint32_t)(q - val_off);
        ++t;
      }
      if (k == nonnull) break;
      if ((k % STR_CK) == 0 && lead) strck[pg.strck_begin + k / STR_CK] = (uint32_t)(q - val_off);
      if (vend - q < 4) { set_err(err, ERR_STRING, p); return; }
      uint32_t l = r.u32(q);
      q += 4;
      if (l > vend - q) { set_err(err, ERR_STRING, p); return; }
      q += l;
    }
    if (ntiles > 0) tiles[pg.tile_begin + ntiles - 1].val_skip = (uint32_t)(q - val_off);
  } else if (enc == E_PLAIN_DICT || enc == E_RLE_DICT) {
    if (pg.dict_page == ~0u) { set_err(err, ERR_DICT_MISSING, p); return; }
    if (nonnull > 0) {
      if (val_len < 1) { set_err(err, ERR_VALUES, p); return; }
      const uint32_t w = r.byte(val_off);
      if (w > 32) { set_err(err, ERR_VALUES, p); return; }
      pg.enc_w = w;
      RunCur c;
      c.next = val_off + 1; c.start = 0; c.n = 0; c.bp = 0; c.val = 0; c.pay = 0; c.hp = val_off + 1;
      bool have = false;
      for (uint32_t t = 0; t < ntiles; ++t) {
        TileDev& tdr = tiles[pg.tile_begin + t];
        const uint32_t k0 = tdr.k0, nnt = tdr.nn;
        for (uint32_t sub = 0; sub < NSUB && sub * SUB_ROWS < nnt; ++sub) {
          const int64_t target = (int64_t)k0 + (int64_t)sub * SUB_ROWS;
          while (!have || c.start + (int64_t)c.n <= target) {
            if (!run_next(r, vend, w, c)) { set_err(err, ERR_VALUES, p); return; }
            have = true;
          }
          if (sub == 0) {
            tdr.val_pos = (uint32_t)(c.hp - val_off);
            tdr.val_skip = (uint32_t)(target - c.start);
          }
          if (lead) ckv[(size_t)(pg.tile_begin + t) * NSUB + sub] = make_ck(c, target, w, val_off + tdr.val_pos);
        }
      }
      while (!have || c.start + (int64_t)c.n < (int64_t)nonnull) {
        if (!run_next(r, vend, w, c)) { set_err(err, ERR_VALUES, p); return; }
        have = true;
      }
    }
  } else if (enc == E_DELTA || (enc == E_DLBA && ch.type == T_BYTE_ARRAY)) {
    // DELTA_BINARY_PACKED values, or the lengths of DELTA_LENGTH_BYTE_ARRAY
    // strings (32-bit), whose chars follow the stream
    bool bad = false;
    uint64_t q = val_off;
    uint64_t B = br_uleb(r, q, vend, bad), M = br_uleb(r, q, vend, bad), total = br_uleb(r, q, vend, bad);
    const int64_t first = unzz(br_uleb(r, q, vend, bad));
    if (bad || B == 0 || B % 128 != 0 || M == 0 || B % M != 0 || (B / M) % 32 != 0 || total != nonnull) {
      set_err(err, ERR_DELTA, p);
      return;
    }
    if (M > 16 || B > 65536) { set_err(err, ERR_UNSUPPORTED, p); return; }
    const uint32_t maxw = ch.type == T_INT64 ? 64 : 32;
    const uint64_t per = B / M;
    pg.enc_w = (uint32_t)B;
    pg.enc_m = (uint32_t)M;
    pg.delta_first = first;
    pg.blocks_at = (uint32_t)(q - val_off);
    // block b holds values [1 + b*B, 1 + (b+1)*B); value 0 is in the header
    const uint64_t nblocks = total > 1 ? (total - 1 + B - 1) / B : 0;
    const bool cached = ntiles <= TC;
    for (uint32_t t = 0; t < ntiles; ++t) {
      tiles[pg.tile_begin + t].val_pos = (uint32_t)(q - val_off);
      tiles[pg.tile_begin + t].val_skip = 0;
      if (cached) {  // every lane wrote every tile above, so each reads its own stores
        s_k0[t] = tiles[pg.tile_begin + t].k0;
        s_nn[t] = tiles[pg.tile_begin + t].nn;
        s_vp[t] = (uint32_t)(q - val_off);
      }
    }
    auto tile_k0 = [&](uint32_t x) { return cached ? s_k0[x] : tiles[pg.tile_begin + x].k0; };
    auto tile_nn = [&](uint32_t x) { return cached ? s_nn[x] : tiles[pg.tile_begin + x].nn; };
    auto tile_vp = [&](uint32_t x) { return cached ? s_vp[x] : tiles[pg.tile_begin + x].val_pos; };
    uint32_t t = 0, ulo = 0;
    for (uint64_t b = 0; b < nblocks; ++b) {
      while (t < ntiles) {
        const uint32_t k0t = tile_k0(t), nnt = tile_nn(t);
        const uint64_t last = (uint64_t)k0t + nnt;  // one past the tile's last value
        if (nnt == 0 || last <= 1) { ++t; continue; }  // needs no block
        const uint64_t first = k0t == 0 ? 1 : k0t;
        const uint64_t nb = (first - 1) / B;
        if (nb != b) break;
        tiles[pg.tile_begin + t].val_pos = (uint32_t)(q - val_off);
        tiles[pg.tile_begin + t].val_skip = (uint32_t)((first - 1) % B);
        if (cached) s_vp[t] = (uint32_t)(q - val_off);
        ++t;
      }
      // this block's header, as checkpoint (b - entry block) of every tile
      // entered so far whose deltas reach block b; tiles before `ulo` end
      // before it
      while (ulo < t) {
        const uint32_t k0u = tile_k0(ulo), nnu = tile_nn(ulo);
        if (nnu != 0 && (uint64_t)k0u + nnu > 1 && ((uint64_t)k0u + nnu - 2) / B >= b) break;
        ++ulo;
      }
      for (uint32_t u = ulo; u < t; ++u) {
        TileDev tu;
        tu.k0 = tile_k0(u);
        tu.nn = tile_nn(u);
        tu.val_pos = tile_vp(u);
        if (tu.nn == 0 || (uint64_t)tu.k0 + tu.nn <= 1) continue;
        const uint64_t fu = tu.k0 == 0 ? 1 : tu.k0;
        const uint64_t bu = (fu - 1) / B;                    // entry block of tile u
        const uint64_t lastb = ((uint64_t)tu.k0 + tu.nn - 2) / B;  // block of its last delta
        if (b >= bu && b <= lastb && b - bu < NSUB && lead)
          ckv[(size_t)(pg.tile_begin + u) * NSUB + (b - bu)] = ck_at(q - val_off - tu.val_pos);
      }
      br_uleb(r, q, vend, bad);  // min delta
      if (bad || M > vend - q) { set_err(err, ERR_DELTA, p); return; }
      const uint64_t left = total - 1 - b * B;  // values from this block on
      const uint64_t used = left < B ? left : B;
      const uint64_t used_mb = (used + per - 1) / per;
      uint64_t body = 0;
      for (uint64_t m = 0; m < used_mb; ++m) {
        const uint32_t w = r.byte(q + m);
        if (w > maxw) { set_err(err, ERR_DELTA, p); return; }
        body += per * w / 8;
      }
      q += M;
      if (body > vend - q) { set_err(err, ERR_DELTA, p); return; }
      q += body;
    }
    pg.chars_at = (uint32_t)(q - val_off);
  }
  pages[p] = pg;
}


// ---------------------------------------------------------------------------
// The index of an open pass.  Every page's streams are found first
// (k_layout); then the chains of its level, index, DELTA or string streams
// are found by one workgroup per page, segment by segment (pq_chain.hpp), and
// what a scan needs is derived from them for all tiles side by side: a tile's
// run is the last one that starts in the last piece with no more rows before
// it, found by a binary search over the pieces.  A page is flagged, and left
// to k_index, when its chain meets an element the grammar does not decode (a
// run header over 32 bits, a payload over LV_PAY bytes), when the chain ends
// early or when an element is malformed.
// ---------------------------------------------------------------------------
constexpr uint32_t LV_PAY = 1024;         // longest payload of a bit-packed level run
constexpr uint32_t LV_SLACK = LV_PAY + 64;

// One thread per page of [p0, p1), dictionary pages or the others.
__global__ void k_layout(uint32_t p0, uint32_t p1, int dicts, PageDev* pages, const PageX* pagex, const ChunkDev* chunks,
                         const uint8_t* file, const uint8_t* scratch, uint32_t* err) {
  const uint32_t p = p0 + blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= p1) return;
  PageDev pg = pages[p];
  if ((pg.kind == PAGE_DICT) != (dicts != 0)) return;
  const int32_t type = chunks[pg.chunk].type;
  const bool optional = chunks[pg.chunk].optional != 0, in_scratch = pg.scratch_len > 0;
  if (pg.kind == PAGE_DICT) {
    pg.val_off = in_scratch ? pg.scratch_off : pg.payload;
    pg.val_len = pg.uncomp_size;
    pg.flags = in_scratch ? 2 : 0;
    pg.dict_maxlen = 0;
    const uint64_t w = type == T_INT32 ? 4 : 8;
    if (type != T_BYTE_ARRAY && (uint64_t)pg.num_values * w > pg.uncomp_size) { set_err(err, ERR_VALUES, p); return; }
    pages[p] = pg;
    return;
  }
  uint64_t def_off = 0, def_len = 0, val_off = 0, val_len = 0;
  if (pg.kind == PAGE_DATA) {
    const uint8_t* base = in_scratch ? scratch : file;
    const uint64_t off = in_scratch ? pg.scratch_off : pg.payload, blen = pg.uncomp_size;
    if (optional) {
      if (blen < 4) { set_err(err, ERR_LEVELS, p); return; }
      const uint64_t n = ld_u32(base, off);
      if (n > blen - 4) { set_err(err, ERR_LEVELS, p); return; }
      def_off = off + 4; def_len = n;
      val_off = off + 4 + n; val_len = blen - 4 - n;
    } else {
      val_off = off; val_len = blen;
    }
    pg.flags = in_scratch ? 3 : 0;
  } else {
    def_off = pg.payload;
    def_len = (uint64_t)pg.def_len;
    if (in_scratch) {
      val_off = pg.scratch_off;
      val_len = pg.scratch_len;
      pg.flags = 2;
    } else {
      val_off = def_off + def_len;
      val_len = pg.comp_size - def_len;
      pg.flags = 0;
    }
  }
  if (pg.encoding == E_DBA && type == T_BYTE_ARRAY && pagex[p].x_total == DBA_UNSUPPORTED) {
    pg.encoding = E_UNDECODED;  // reported by the decode kernels when the column is scanned
  } else if (pg.encoding == E_DBA && type == T_BYTE_ARRAY) {
    // DELTA_BYTE_ARRAY: the values, expanded to the PLAIN layout by k_dba,
    // are indexed and decoded like a PLAIN page
    val_off = pagex[p].x_off;
    val_len = pagex[p].xlen;
    pg.flags = (uint8_t)((pg.flags & 1) | 4);
  }
  pg.def_off = def_off;
  pg.def_len = (int32_t)def_len;
  pg.val_off = val_off;
  pg.val_len = (uint32_t)val_len;
  pages[p] = pg;
}

// A run of a w-bit hybrid stream from its first eight bytes, left stream
// bytes from its header on (run_next's rules; headers of at most 28 bits and
// payloads below 2^24 groups, STEP_ODD otherwise).  The chain kernels decode one
// at every byte of a stream, so instructions count.
struct HRun {
  uint32_t adv;  // its bytes, or STEP_BAD / STEP_ODD
  uint32_t hl;   // header bytes
  uint32_t n;    // values
  uint32_t val;  // RLE, w <= 8: the value
  bool bp;
};
__device__ __forceinline__ HRun hrun(uint32_t lo, uint32_t hi, uint32_t left, uint32_t w) {
  HRun r;
  const uint32_t cont = ~lo & 0x80808080u;  // bytes that end the header
  const uint32_t h4 = (lo & 0x7fu) | ((lo >> 1) & 0x3f80u) | ((lo >> 2) & 0x1fc000u) | ((lo >> 3) & 0xfe00000u);
  r.hl = ((uint32_t)__builtin_ctz(cont | 0x80000000u) >> 3) + 1;
  const uint32_t h = __builtin_amdgcn_ubfe(h4, 0, 7 * r.hl), g = h >> 1;
  r.bp = (h & 1) != 0;
  const uint32_t pay = r.bp ? __umul24(g, w) : (w + 7) / 8;
  r.n = r.bp ? 8 * g : g;
  r.val = (r.hl < 4 ? __builtin_amdgcn_alignbyte(hi, lo, r.hl) : hi) & 0xffu;
  r.adv = cont == 0 || (r.bp && (g >> 24)) ? STEP_ODD : r.hl + pay > left ? STEP_BAD : r.hl + pay;
  return r;
}
// A level run: levels are 0 or 1.
__device__ __forceinline__ HRun lrun(uint32_t lo, uint32_t hi, uint32_t left) {
  HRun r = hrun(lo, hi, left, 1);
  if (!r.bp && r.val > 1 && r.adv != STEP_ODD) r.adv = STEP_BAD;
  return r;
}

// A stream of a page as the chain kernels read it: bytes [m, m + len) of a
// 16-byte aligned base, readable up to lim (a multiple of 16).
struct ChainSrc {
  const uint8_t* base;
  uint32_t m, len, lim;
};
__device__ __forceinline__ ChainSrc chain_src(const uint8_t* buf, uint64_t buflim, uint64_t off, uint64_t len) {
  ChainSrc c;
  c.m = (uint32_t)(off & 15);
  c.base = buf + (off - c.m);
  c.len = (uint32_t)len;
  c.lim = (uint32_t)min(buflim - (off - c.m), (uint64_t)((c.m + c.len + 64 + 15) & ~15u));
  return c;
}
__device__ __forceinline__ ChainSrc level_src(const PageDev& pg, const OpenBufs& b) {
  const bool sc = (pg.flags & 1) != 0;
  return chain_src(sc ? b.scratch : b.file, sc ? b.scratch_lim : b.file_lim, pg.def_off, pg.def_len > 0 ? pg.def_len : 0);
}
// from byte `from` of the value stream on
__device__ __forceinline__ ChainSrc value_src(const PageDev& pg, const OpenBufs& b, uint32_t from) {
  const uint8_t* buf = (pg.flags & 4) ? b.xscratch : ((pg.flags & 2) ? b.scratch : b.file);
  const uint64_t lim = (pg.flags & 4) ? b.xscratch_lim : ((pg.flags & 2) ? b.scratch_lim : b.file_lim);
  return chain_src(buf, lim, pg.val_off + from, pg.val_len > from ? pg.val_len - from : 0);
}

// Exclusive prefix sum over the workgroup (and the total).
template <uint32_t NT>
__device__ __forceinline__ uint32_t wg_scan(uint32_t v, uint32_t* s_sum, uint32_t& total) {
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t incl = wave_incl_scan_u32(v);
  if (lane == 63) s_sum[wave] = incl;
  __syncthreads();
  uint32_t before = incl - v;
  total = 0;
#pragma unroll
  for (uint32_t w = 0; w < NT / 64; ++w) {
    const uint32_t x = s_sum[w];
    if (w < wave) before += x;
    total += x;
  }
  return before;
}
template <uint32_t NT>
__device__ __forceinline__ uint64_t wg_scan64(uint64_t v, uint64_t* s_sum, uint64_t& total) {
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t incl = wave_incl_scan_u64(v);
  if (lane == 63) s_sum[wave] = incl;
  __syncthreads();
  uint64_t before = incl - v;
  total = 0;
#pragma unroll
  for (uint32_t w = 0; w < NT / 64; ++w) {
    const uint64_t x = s_sum[w];
    if (w < wave) before += x;
    total += x;
  }
  return before;
}
__device__ __forceinline__ uint32_t sat32(uint64_t v) { return v > 0xffffffffull ? 0xffffffffu : (uint32_t)v; }

// ---------------------------------------------------------------------------
// k_levels: the runs of a page's definition levels, one workgroup per page:
// rows and valid rows before every piece, and the page's non-null count.
// What bounds it: the vector instructions that decode a run at every byte.
// Measured on a 4M-row wide table in 1M-row row groups and 1 MiB pages, with
// k_tiles: 0.24 + 0.16 ms; one wave per 2 KiB segment whose first lane walks the
// runs, after 128 candidate walks per segment: 1.18 + 1.52 ms.
// ---------------------------------------------------------------------------
template <uint32_t NT>
__global__ __launch_bounds__(NT) void k_levels(const IxPage* ixs, const uint32_t* list, PageDev* pages, OpenBufs bufs,
                                               uint32_t* at, uint32_t* val, uint8_t* ent, uint32_t* flag,
                                               const uint32_t* err) {
  __shared__ ChainLds<NT, LV_SLACK> L;
  __shared__ uint64_t s_rows[NT / 64];
  __shared__ uint32_t s_val[NT / 64];
  if (*(const volatile uint32_t*)err != 0) return;
  const uint32_t ixi = list[blockIdx.x], tid = threadIdx.x;
  const IxPage ix = ixs[ixi];
  const ChainSrc st = level_src(pages[ix.page], bufs);
  const uint64_t nv = (uint64_t)pages[ix.page].num_values;
  const uint32_t iend = st.m + st.len;
  uint32_t ip = st.m, wz = 0, valid = 0;
  uint64_t rows = 0;
  bool odd = false;
  auto step = [](uint32_t lo, uint32_t hi, uint32_t left, uint32_t) -> uint32_t { return lrun(lo, hi, left).adv; };
  // set bits among the first k values of a payload from segment byte o
  auto pop = [&](uint32_t o, uint32_t k) -> uint32_t {
    uint32_t c = 0;
    for (uint32_t i = 0; 8 * i < k; i += 4) {
      uint32_t v = __builtin_amdgcn_alignbyte(L.in[((o + i) >> 2) + 1], L.in[(o + i) >> 2], (o + i) & 3);
      const uint32_t left = k - 8 * i;
      if (left < 32) v &= (1u << left) - 1u;
      c += __popc(v);
    }
    return c;
  };
  while (ip < iend && rows < nv) {
    const uint32_t S = ip & ~(CH_PIECE - 1);
    for (uint32_t w = wz + tid; w < min(S / CH_PIECE, ix.nlv); w += NT) {
      at[ix.lv0 + w] = sat32(rows);
      val[ix.lv0 + w] = valid;
      ent[ix.lv0 + w] = CH_NONE;
    }
    uint32_t code;
    const uint32_t next = L.find(step, st.base, st.lim, S, ip, iend, code);
    const uint32_t plen = L.piece_len(S, iend), y0 = tid * CH_PIECE, pe = L.pent[tid];
    uint64_t cnt = 0;
    uint32_t v = 0;
    bool big = false;
    for (uint32_t y = pe; y < plen;) {
      uint32_t lo, hi;
      L.bytes8(y0 + y, lo, hi);
      const HRun r = lrun(lo, hi, iend - S - y0 - y);
      if (r.adv == STEP_BAD || r.adv == STEP_ODD) break;
      if (!r.bp) v += r.val * r.n;
      else if (r.n <= 8 * LV_PAY) v += pop(y0 + y + r.hl, r.n);
      else big = true;
      cnt += r.n;
      y += r.adv;
    }
    uint64_t tot;
    uint32_t vtot;
    const uint64_t start = rows + wg_scan64<NT>(cnt, s_rows, tot);
    const uint32_t vstart = valid + wg_scan<NT>(v, s_val, vtot);
    const uint32_t pc = S / CH_PIECE + tid;
    if (pc < ix.nlv) {
      at[ix.lv0 + pc] = sat32(start);
      val[ix.lv0 + pc] = vstart;
      ent[ix.lv0 + pc] = (uint8_t)pe;
    }
    odd |= big && start < nv;
    if (start < nv && start + cnt >= nv) {  // the run covering the last row
      uint64_t r0 = start;
      uint32_t vv = vstart;
      for (uint32_t y = pe; y < plen;) {
        uint32_t lo, hi;
        L.bytes8(y0 + y, lo, hi);
        const HRun r = lrun(lo, hi, iend - S - y0 - y);
        const bool last = r0 + r.n >= nv;
        const uint32_t n = last ? (uint32_t)(nv - r0) : r.n;
        vv += !r.bp ? r.val * n : (r.n <= 8 * LV_PAY ? pop(y0 + y + r.hl, n) : 0u);
        if (last) break;
        r0 += r.n;
        y += r.adv;
      }
      pages[ix.page].nonnull = vv;
    }
    wz = S / CH_PIECE + NT;
    rows += tot;
    valid += vtot;
    ip = next;
    if (code) break;
  }
  for (uint32_t w = wz + tid; w < ix.nlv; w += NT) {
    at[ix.lv0 + w] = 0xffffffffu;
    ent[ix.lv0 + w] = CH_NONE;
  }
  if (__syncthreads_or(odd) || rows < nv)
    if (tid == 0) flag[ixi] = 1;
}

// The last page of ixs[0, nix) whose first tile is at or before t.
__device__ __forceinline__ uint32_t ix_of_tile(const IxPage* ixs, uint32_t nix, uint32_t t) {
  uint32_t lo = 0, hi = nix;
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) >> 1;
    if (ixs[mid].tile0 <= t) lo = mid; else hi = mid;
  }
  return lo;
}
// The last of n pieces with at most v rows (values) before it.
__device__ __forceinline__ uint32_t piece_of(const uint32_t* at, uint32_t n, uint32_t v) {
  uint32_t lo = 0, hi = n;
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) >> 1;
    if (at[mid] <= v) lo = mid; else hi = mid;
  }
  return lo;
}

// Bytes of one piece and those after it in the lane's LDS row (13 dwords: no
// bank conflicts).
constexpr uint32_t ROW_DW = 13;
__device__ __forceinline__ void row_load(uint32_t* row, const ChainSrc& st, uint32_t piece) {
#pragma unroll
  for (uint32_t k = 0; k < 3; ++k) {
    const uint32_t q = piece * CH_PIECE + 16 * k;
    u32x4c v = {0u, 0u, 0u, 0u};
    if (q < st.lim) v = *reinterpret_cast<const u32x4c*>(st.base + q);
    row[4 * k] = v.x; row[4 * k + 1] = v.y; row[4 * k + 2] = v.z; row[4 * k + 3] = v.w;
  }
}
__device__ __forceinline__ void row_bytes8(const uint32_t* row, uint32_t y, uint32_t& lo, uint32_t& hi) {
  const uint32_t j = y >> 2, w0 = row[j], w1 = row[j + 1], w2 = row[j + 2];
  lo = __builtin_amdgcn_alignbyte(w1, w0, y & 3);
  hi = __builtin_amdgcn_alignbyte(w2, w1, y & 3);
}
// The run holding value v: the runs of piece pc from byte y on, the first of
// them at value r; positions relative to the stream's first byte.
__device__ __forceinline__ RunCur row_run(const uint32_t* row, const ChainSrc& st, uint32_t pc, uint32_t y, uint64_t r,
                                          uint64_t v, uint32_t w, bool& found) {
  RunCur c;
  c.hp = c.next = c.pay = 0; c.start = 0; c.n = 0; c.bp = 0; c.val = 0;
  found = false;
  while (y < CH_PIECE) {
    uint32_t lo, hi;
    row_bytes8(row, y, lo, hi);
    const uint32_t q = pc * CH_PIECE + y, iend = st.m + st.len;
    const HRun h = hrun(lo, hi, q < iend ? iend - q : 0u, w);
    if (h.adv == STEP_BAD || h.adv == STEP_ODD) break;
    if (v < r + h.n) {
      c.hp = q - st.m;
      c.pay = c.hp + h.hl;
      c.next = c.hp + h.adv;
      c.start = (int64_t)r;
      c.n = h.n;
      c.bp = h.bp ? 1 : 0;
      c.val = h.val;
      found = true;
      break;
    }
    r += h.n;
    y += h.adv;
  }
  return c;
}

// ---------------------------------------------------------------------------
// k_tiles: one wave per tile: its entry in the level stream, the values before
// it, and its level checkpoints, lane k's from the run of row 16 k.  What bounds
// it: the dependent loads of the two binary searches.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_tiles(const IxPage* ixs, uint32_t nix, uint32_t tile0, uint32_t ntiles,
                                               const PageDev* pages, const ChunkDev* chunks, OpenBufs bufs,
                                               const uint32_t* at, const uint32_t* val, const uint8_t* ent,
                                               const uint32_t* flag, TileDev* tiles, uint32_t* ckl, Ck* ckv,
                                               const uint32_t* err) {
  __shared__ uint32_t s_row[256][ROW_DW];
  if (*(const volatile uint32_t*)err != 0) return;
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t i = (uint32_t)__builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (threadIdx.x >> 6)));
  if (i >= ntiles) return;
  const uint32_t T = tile0 + i;
  const uint32_t ixi = ix_of_tile(ixs, nix, T);
  const IxPage ix = ixs[ixi];
  if (flag[ixi] || T - ix.tile0 >= ix.ntiles) return;
  const PageDev& pg = pages[ix.page];
  const uint32_t R0 = (T - ix.tile0) * TILE_ROWS;
  TileDev td;
  td.page = ix.page;
  td.row0 = R0;
  td.k0 = R0;
  td.nn = 0;
  td.def_pos = 0; td.def_skip = 0; td.val_pos = 0; td.val_skip = 0;
  if (lane < NSUB) ckv[(size_t)T * NSUB + lane] = ck_none();
  if (!chunks[pg.chunk].optional) {
    ckl[(size_t)T * NLCK + lane] = LCK_NONE;
    if (lane == 0) tiles[T] = td;
    return;
  }
  const ChainSrc st = level_src(pg, bufs);
  const uint32_t nv = (uint32_t)pg.num_values, row = R0 + lane * LROWS;
  const bool live = row < nv;
  const uint32_t v = live ? row : R0;
  const uint32_t pc = piece_of(at + ix.lv0, ix.nlv, v);
  uint32_t* rowp = &s_row[threadIdx.x][0];
  row_load(rowp, st, pc);
  bool found;
  const RunCur c = row_run(rowp, st, pc, ent[ix.lv0 + pc], at[ix.lv0 + pc], v, 1, found);
  const uint32_t entry = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)c.hp);
  ckl[(size_t)T * NLCK + lane] = live && found ? make_lck(c, (int64_t)row, entry) : LCK_NONE;
  if (lane == 0) {
    // valid rows before the tile: those before the piece, of the piece's runs
    // before the tile's and of that run before the tile
    auto pop = [&](uint64_t pay, uint64_t k) -> uint32_t {
      uint32_t s = 0;
      for (uint64_t b = 0; b < k; b += 32) {
        uint32_t x = ld_u32(st.base, st.m + pay + (b >> 3));
        if (k - b < 32) x &= (1u << (k - b)) - 1u;
        s += __popc(x);
      }
      return s;
    };
    uint32_t k0 = val[ix.lv0 + pc];
    for (uint32_t y = ent[ix.lv0 + pc]; y < CH_PIECE && pc * CH_PIECE + y - st.m < c.hp;) {
      uint32_t lo, hi;
      row_bytes8(rowp, y, lo, hi);
      const HRun h = hrun(lo, hi, st.m + st.len - (pc * CH_PIECE + y), 1);
      k0 += h.bp ? pop((uint64_t)pc * CH_PIECE + y - st.m + h.hl, h.n) : h.val * h.n;
      y += h.adv;
    }
    const uint32_t skip = R0 - (uint32_t)c.start;
    k0 += c.bp ? pop(c.pay, skip) : c.val * skip;
    td.k0 = k0;
    td.def_pos = (uint32_t)c.hp;
    td.def_skip = skip;
    tiles[T] = td;
  }
}

// ---------------------------------------------------------------------------
// k_values: one thread per data page, after its levels: the checks of its value
// stream's header and the facts the later kernels read from it.
// ---------------------------------------------------------------------------
__global__ void k_values(const IxPage* ixs, uint32_t nix, PageDev* pages, const PageX* pagex, const ChunkDev* chunks,
                         OpenBufs bufs, const uint32_t* flag, uint32_t* err) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nix || flag[i]) return;
  const uint32_t p = ixs[i].page;
  PageDev& pg = pages[p];
  if (pg.kind == PAGE_DICT) return;
  const ChunkDev& ch = chunks[pg.chunk];
  const uint32_t nv = pg.num_values > 0 ? (uint32_t)pg.num_values : 0u;
  if (!ch.optional || nv == 0) pg.nonnull = nv;
  const uint32_t nonnull = pg.nonnull;
  if (pg.kind == PAGE_DATA_V2 && (int64_t)pg.num_nulls != (int64_t)nv - (int64_t)nonnull) { set_err(err, ERR_V2, p); return; }
  const int enc = pg.encoding;
  const uint8_t* vbase = (pg.flags & 4) ? bufs.xscratch : ((pg.flags & 2) ? bufs.scratch : bufs.file);
  const uint64_t val_off = pg.val_off, val_len = pg.val_len;
  if ((enc == E_PLAIN || enc == E_BSS) && ch.type != T_BYTE_ARRAY) {
    const uint64_t w = ch.type == T_INT32 ? 4 : 8;
    if ((uint64_t)nonnull * w > val_len) set_err(err, ERR_VALUES, p);
  } else if (enc == E_DBA) {
    if (pagex[p].x_total != nonnull) set_err(err, ERR_VALUES, p);
  } else if (enc == E_PLAIN_DICT || enc == E_RLE_DICT) {
    if (pg.dict_page == ~0u) { set_err(err, ERR_DICT_MISSING, p); return; }
    if (nonnull > 0) {
      if (val_len < 1) { set_err(err, ERR_VALUES, p); return; }
      const uint32_t w = vbase[val_off];
      if (w > 32) { set_err(err, ERR_VALUES, p); return; }
      pg.enc_w = w;
    }
  } else if (enc == E_DELTA || (enc == E_DLBA && ch.type == T_BYTE_ARRAY)) {
    BR r;
    r.init(vbase);
    bool bad = false;
    uint64_t q = val_off;
    const uint64_t vend = val_off + val_len;
    const uint64_t B = br_uleb(r, q, vend, bad), M = br_uleb(r, q, vend, bad), total = br_uleb(r, q, vend, bad);
    const int64_t first = unzz(br_uleb(r, q, vend, bad));
    if (bad || B == 0 || B % 128 != 0 || M == 0 || B % M != 0 || (B / M) % 32 != 0 || total != nonnull) {
      set_err(err, ERR_DELTA, p);
      return;
    }
    if (M > 16 || B > 65536) { set_err(err, ERR_UNSUPPORTED, p); return; }
    pg.enc_w = (uint32_t)B;
    pg.enc_m = (uint32_t)M;
    pg.delta_first = first;
    pg.blocks_at = (uint32_t)(q - val_off);
    pg.chars_at = pg.blocks_at;  // (a stream without blocks; else stored by k_dl)
  }
}

// ---------------------------------------------------------------------------
// k_strings: the (u32 length, bytes) chain of a PLAIN string page, an expanded
// DELTA_BYTE_ARRAY page or a string dictionary, one workgroup per page: the
// position of every STR_CK-th value, and a dictionary's longest entry.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t str_step(uint32_t lo, uint32_t left) {
  return left < 4 || lo > left - 4 ? STEP_BAD : 4 + lo;
}
__device__ __forceinline__ uint32_t str_count(const PageDev& pg) {
  return pg.kind == PAGE_DICT ? (pg.num_values > 0 ? (uint32_t)pg.num_values : 0u) : pg.nonnull;
}

template <uint32_t NT>
__global__ __launch_bounds__(NT) void k_strings(const IxPage* ixs, const uint32_t* list, PageDev* pages, OpenBufs bufs,
                                                uint32_t* strck, uint32_t* flag, const uint32_t* err,
                                                const uint32_t* seq) {
  __shared__ ChainLds<NT, 64> L;
  __shared__ uint32_t s_sum[NT / 64];
  __shared__ uint32_t s_max;
  const uint32_t ixi = list[blockIdx.x], tid = threadIdx.x;
  if (*(const volatile uint32_t*)err != 0 || flag[ixi]) return;
  if (seq && !seq[blockIdx.x]) return;  // (a page whose segments the k_seg kernels did)
  const uint32_t p = ixs[ixi].page;
  PageDev& pg = pages[p];
  const bool dict = pg.kind == PAGE_DICT;
  const uint32_t n = str_count(pg);
  const ChainSrc st = value_src(pg, bufs, 0);
  uint32_t* ck = strck + pg.strck_begin;
  const uint32_t iend = st.m + st.len;
  uint32_t ip = st.m, k = 0, maxlen = 0;
  if (long_strings(st.len, n)) {
    if (tid != 0) return;
    while (k < n && iend - ip >= 4) {
      const uint32_t len = ld_u32(st.base, ip);
      if (len > iend - ip - 4) break;
      if (k % STR_CK == 0) ck[k / STR_CK] = ip - st.m;
      maxlen = max(maxlen, len);
      ip += 4 + len;
      ++k;
    }
    if (dict) pg.dict_maxlen = maxlen;
    if (k < n) flag[ixi] = 1;
    return;
  }
  if (tid == 0) s_max = 0;
  auto step = [](uint32_t lo, uint32_t, uint32_t left, uint32_t) -> uint32_t { return str_step(lo, left); };
  while (ip < iend && k < n) {
    const uint32_t S = ip & ~(CH_PIECE - 1);
    uint32_t code;
    const uint32_t next = L.find(step, st.base, st.lim, S, ip, iend, code);
    const uint32_t plen = L.piece_len(S, iend), y0 = tid * CH_PIECE;
    uint32_t mask = 0, lens[CH_PIECE / 4];
    uint32_t cnt = 0;
#pragma unroll
    for (uint32_t j = 0; j < CH_PIECE / 4; ++j) lens[j] = 0;
    uint32_t y = L.pent[tid];
#pragma unroll
    for (uint32_t j = 0; j < CH_PIECE / 4; ++j) {  // (each takes four bytes or more)
      if (y < plen) {
        uint32_t lo, hi;
        L.bytes8(y0 + y, lo, hi);
        const uint32_t a = step(lo, hi, iend - S - y0 - y, 0);
        if (a == STEP_BAD) {
          y = CH_PIECE;
        } else {
          mask |= 1u << y;
          lens[j] = lo;
          y += a;
          ++cnt;
        }
      }
    }
    uint32_t tot;
    const uint32_t k0 = k + wg_scan<NT>(cnt, s_sum, tot);
    const uint32_t have = k0 < n ? min(cnt, n - k0) : 0u;  // those of the page's n values
#pragma unroll
    for (uint32_t j = 0; j < CH_PIECE / 4; ++j)
      if (j < have) maxlen = max(maxlen, lens[j]);
    uint32_t at = (STR_CK - k0 % STR_CK) % STR_CK;  // the piece's element at a checkpoint
    if (at < have) {
      for (uint32_t m = mask;; m &= m - 1, --at)
        if (at == 0) {
          ck[(k0 + STR_CK - 1) / STR_CK] = S + y0 + (uint32_t)__builtin_ctz(m) - st.m;
          break;
        }
    }
    k += tot;  // (at most 2^31: four bytes each)
    ip = next;
    if (code) break;
  }
  if (dict) {
    __syncthreads();
    if (maxlen) atomicMax(&s_max, maxlen);
    __syncthreads();
    if (tid == 0) pg.dict_maxlen = s_max;
  }
  if (tid == 0 && k < n) flag[ixi] = 1;
}

// ---------------------------------------------------------------------------
// k_di: the runs of a page's dictionary indices, one workgroup per page: the
// values before every piece.  Measured on the 4M-row wide table (pages of up to
// 1 MiB, 32 segments in a row): 0.66 ms; up to 1,024 candidate walks per segment, a
// link and one wave per segment: 1.4 ms.
// ---------------------------------------------------------------------------
template <uint32_t NT>
__global__ __launch_bounds__(NT) void k_di(const IxPage* ixs, const uint32_t* list, const PageDev* pages, OpenBufs bufs,
                                           uint32_t* at, uint8_t* ent, uint32_t* flag, const uint32_t* err,
                                           const uint32_t* seq) {
  __shared__ ChainLds<NT, 64> L;
  __shared__ uint64_t s_sum[NT / 64];
  const uint32_t ixi = list[blockIdx.x], tid = threadIdx.x;
  if (*(const volatile uint32_t*)err != 0 || flag[ixi]) return;
  if (seq && !seq[blockIdx.x]) return;
  const IxPage ix = ixs[ixi];
  const PageDev& pg = pages[ix.page];
  const uint64_t n = pg.nonnull;
  if (n == 0) return;
  const uint32_t w = pg.enc_w;
  const ChainSrc st = value_src(pg, bufs, 1);
  const uint32_t iend = st.m + st.len;
  uint32_t ip = st.m, wz = 0;
  uint64_t k = 0;
  auto step = [w](uint32_t lo, uint32_t hi, uint32_t left, uint32_t) -> uint32_t { return hrun(lo, hi, left, w).adv; };
  while (ip < iend && k < n) {
    const uint32_t S = ip & ~(CH_PIECE - 1);
    for (uint32_t x = wz + tid; x < min(S / CH_PIECE, ix.nv); x += NT) {
      at[ix.v0 + x] = sat32(k);
      ent[ix.v0 + x] = CH_NONE;
    }
    uint32_t code;
    const uint32_t next = L.find(step, st.base, st.lim, S, ip, iend, code);
    const uint32_t plen = L.piece_len(S, iend), y0 = tid * CH_PIECE, pe = L.pent[tid];
    uint64_t cnt = 0;
    for (uint32_t y = pe; y < plen;) {
      uint32_t lo, hi;
      L.bytes8(y0 + y, lo, hi);
      const HRun r = hrun(lo, hi, iend - S - y0 - y, w);
      if (r.adv == STEP_BAD || r.adv == STEP_ODD) break;
      cnt += r.n;
      y += r.adv;
    }
    uint64_t tot;
    const uint64_t k0 = k + wg_scan64<NT>(cnt, s_sum, tot);
    const uint32_t pc = S / CH_PIECE + tid;
    if (pc < ix.nv) {
      at[ix.v0 + pc] = sat32(k0);
      ent[ix.v0 + pc] = (uint8_t)pe;
    }
    wz = S / CH_PIECE + NT;
    k += tot;
    ip = next;
    if (code) break;
  }
  for (uint32_t x = wz + tid; x < ix.nv; x += NT) {
    at[ix.v0 + x] = 0xffffffffu;
    ent[ix.v0 + x] = CH_NONE;
  }
  if (tid == 0 && k < n) flag[ixi] = 1;
}

// ---------------------------------------------------------------------------
// k_dl: the blocks of a page's DELTA_BINARY_PACKED values (or of the lengths of
// a DELTA_LENGTH_BYTE_ARRAY page), one workgroup per page: every block's
// position and the stream's end.  Every block is taken as a full one; the
// last holds only the miniblocks its values use, whose end follows from its
// header.
// ---------------------------------------------------------------------------
template <class L>
struct DlBlocks {
  const L* lds;
  uint32_t M, per, maxw;
  // bytes of the block at segment byte y whose first `used` miniblocks are
  // stored (STEP_BAD: malformed)
  __device__ __forceinline__ uint32_t len(uint32_t lo, uint32_t hi, uint32_t left, uint32_t y, uint32_t used) const {
    const uint32_t c0 = ~lo & 0x80808080u, c1 = ~hi & 0x80808080u;
    uint32_t hl;  // bytes of the minimum delta
    if (c0) hl = ((uint32_t)__builtin_ctz(c0) >> 3) + 1;
    else if (c1) hl = ((uint32_t)__builtin_ctz(c1) >> 3) + 5;
    else if (!(lds->byte(y + 8) & 0x80)) hl = 9;
    else if (lds->byte(y + 9) <= 1) hl = 10;
    else return STEP_BAD;
    if (hl > left || M > left - hl) return STEP_BAD;
    uint32_t body = 0;
    bool wide = false;
    for (uint32_t m = 0; m < used; ++m) {
      const uint32_t w = lds->byte(y + hl + m);
      wide |= w > maxw;
      body += per / 8 * w;
    }
    return wide || body > left - hl - M ? STEP_BAD : hl + M + body;
  }
  __device__ __forceinline__ uint32_t operator()(uint32_t lo, uint32_t hi, uint32_t left, uint32_t y) const {
    return len(lo, hi, left, y, M);
  }
};
__device__ __forceinline__ uint32_t dl_nblocks(const PageDev& pg) {
  return pg.nonnull > 1 ? (uint32_t)(((uint64_t)pg.nonnull - 1 + pg.enc_w - 1) / pg.enc_w) : 0u;
}
// miniblocks of block b that hold values
__device__ __forceinline__ uint32_t dl_used(const PageDev& pg, uint32_t b) {
  const uint64_t left = (uint64_t)pg.nonnull - 1 - (uint64_t)b * pg.enc_w;
  const uint32_t per = pg.enc_w / pg.enc_m;
  return (uint32_t)((min(left, (uint64_t)pg.enc_w) + per - 1) / per);
}

template <uint32_t NT>
__global__ __launch_bounds__(NT) void k_dl(const IxPage* ixs, const uint32_t* list, PageDev* pages,
                                           const ChunkDev* chunks, OpenBufs bufs, uint32_t* blkpos, uint32_t* flag,
                                           const uint32_t* err, const uint32_t* seq) {
  __shared__ ChainLds<NT, 64> L;
  __shared__ uint32_t s_sum[NT / 64];
  const uint32_t ixi = list[blockIdx.x], tid = threadIdx.x;
  if (*(const volatile uint32_t*)err != 0 || flag[ixi]) return;
  if (seq && !seq[blockIdx.x]) return;
  const IxPage ix = ixs[ixi];
  PageDev& pg = pages[ix.page];
  const uint32_t nblocks = dl_nblocks(pg);
  if (nblocks == 0) return;
  const DlBlocks<ChainLds<NT, 64>> step{&L, pg.enc_m, pg.enc_w / pg.enc_m, chunks[pg.chunk].type == T_INT64 ? 64u : 32u};
  const ChainSrc st = value_src(pg, bufs, pg.blocks_at);
  const uint32_t iend = st.m + st.len;
  uint32_t ip = st.m, k = 0;
  bool bad = false;
  while (ip < iend && k < nblocks) {
    const uint32_t S = ip & ~(CH_PIECE - 1);
    uint32_t code;
    const uint32_t next = L.find(step, st.base, st.lim, S, ip, iend, code);
    const uint32_t plen = L.piece_len(S, iend), y0 = tid * CH_PIECE;
    uint32_t mask = 0;
    for (uint32_t y = L.pent[tid]; y < plen;) {
      uint32_t lo, hi;
      mask |= 1u << y;
      L.bytes8(y0 + y, lo, hi);
      const uint32_t a = step(lo, hi, iend - S - y0 - y, y0 + y);
      if (a == STEP_BAD) break;
      y += a;
    }
    uint32_t tot;
    uint32_t b = k + wg_scan<NT>((uint32_t)__popc(mask), s_sum, tot);
    for (uint32_t m = mask; m && b < nblocks; m &= m - 1, ++b) {
      const uint32_t y = y0 + (uint32_t)__builtin_ctz(m), q = S + y - st.m;
      blkpos[ix.v0 + b] = pg.blocks_at + q;
      if (b + 1 == nblocks) {
        uint32_t lo, hi;
        L.bytes8(y, lo, hi);
        const uint32_t a = step.len(lo, hi, iend - S - y, y, dl_used(pg, b));
        if (a == STEP_BAD) bad = true;
        else pg.chars_at = pg.blocks_at + q + a;
      }
    }
    k += tot;
    ip = next;
    if (code) break;
  }
  if (__syncthreads_or(bad) || k < nblocks)
    if (tid == 0) flag[ixi] = 1;
}

// ---------------------------------------------------------------------------
// The segments of long value streams side by side, where a pass has too few
// pages to fill the chip with one workgroup each (above all the dictionaries
// of high-cardinality string columns, tens of MiB); F: SEG_STR, SEG_DI, SEG_DL.
//   k_seg_cand  where the chain from each of a segment's first 1,024 or 2,048 bytes
//               leaves the segment;
//   k_seg_link  the true chain's entry into every segment, one workgroup per
//               page, 64 segments at a time (the exits of their first 64 bytes in
//               LDS): through 8 groups of 8 segments from every candidate side
//               by side, from group to group, then through each group; where a
//               chain leaves the candidates in LDS one thread follows it.  A page
//               whose chain enters a segment past all candidates is left to the
//               one-workgroup kernel;
//   k_seg_fill  values (blocks) before every piece, within the segment;
//   k_seg_base  values (blocks) before every segment;
//   k_str_ck, k_dl_ck  string checkpoints and block positions, one thread per
//               piece.
// A segment's exits are found twice, so with a page for every CU the
// one-workgroup kernels are faster; the choice is made on the host.
// Measured on the 4M-row wide table in 1M-row row groups: four string dictionaries of
// 17.7 MB 0.45 ms (0.58 ms with one thread that links all segments of a page in
// turn: k_seg_link 170, now 32 us; k_strings 10.9 ms, 540 segments in a row at 20 us; candidate walks
// of 64 lanes per segment, a thread that links them and a second walk 1.2 ms),
// the index streams of nine columns 0.38 ms (k_di 0.66 ms), one DELTA column 0.12 ms
// (k_dl 0.53 ms).
// ---------------------------------------------------------------------------
using SegLds = ChainLds<1024, 64>;
constexpr uint32_t SEG_NT = 1024, SEG_BYTES = SEG_NT * CH_PIECE;
// Candidates per segment (their exits SEG_CAND apart): 63 groups of 32-bit
// indices, the longest run of the usual writers, take 2,017 bytes.
constexpr uint32_t SEG_CAND = 2048;
template <int F>
constexpr uint32_t seg_cands() { return F == SEG_DI ? SEG_CAND : SEG_NT; }
static_assert(SEG_CAND <= SegLds::REG, "candidates: within the first region");

template <int F>
__device__ __forceinline__ ChainSrc seg_src(const PageDev& pg, const OpenBufs& bufs) {
  return value_src(pg, bufs, F == SEG_STR ? 0u : F == SEG_DI ? 1u : pg.blocks_at);
}
template <int F>
struct SegStep {
  DlBlocks<SegLds> dl;
  uint32_t w;
  __device__ __forceinline__ SegStep(const SegLds* L, const PageDev& pg, const ChunkDev* chunks) {
    w = pg.enc_w;
    if (F == SEG_DL) dl = DlBlocks<SegLds>{L, pg.enc_m, pg.enc_w / pg.enc_m, chunks[pg.chunk].type == T_INT64 ? 64u : 32u};
  }
  __device__ __forceinline__ uint32_t operator()(uint32_t lo, uint32_t hi, uint32_t left, uint32_t y) const {
    if constexpr (F == SEG_STR) return str_step(lo, left);
    else if constexpr (F == SEG_DI) return hrun(lo, hi, left, w).adv;
    else return dl(lo, hi, left, y);
  }
};
// values (blocks) the page needs from the chain
template <int F>
__device__ __forceinline__ uint32_t seg_need(const PageDev& pg) {
  return F == SEG_STR ? str_count(pg) : F == SEG_DI ? pg.nonnull : dl_nblocks(pg);
}

template <int F>
__global__ __launch_bounds__(SEG_NT) void k_seg_cand(const IxPage* ixs, const SegPage* sps, const uint32_t* seg_sp,
                                                     const PageDev* pages, const ChunkDev* chunks, OpenBufs bufs,
                                                     uint32_t* exits, const uint32_t* flag, const uint32_t* err) {
  __shared__ SegLds L;
  const SegPage sp = sps[seg_sp[blockIdx.x]];
  if (*(const volatile uint32_t*)err != 0 || flag[sp.ix]) return;
  const PageDev& pg = pages[ixs[sp.ix].page];
  if (seg_need<F>(pg) == 0) return;
  const ChainSrc st = seg_src<F>(pg, bufs);
  const uint32_t S = (blockIdx.x - sp.seg0) * SEG_BYTES, iend = st.m + st.len;
  if (S >= iend) return;
  const SegStep<F> step(&L, pg, chunks);
  L.exits(step, st.base, st.lim, S, iend);
  for (uint32_t c = threadIdx.x; c < seg_cands<F>(); c += SEG_NT)
    exits[(size_t)blockIdx.x * SEG_CAND + c] = L.follow(step, c, S, iend);
}

template <int F>
__global__ __launch_bounds__(256) void k_seg_link(const IxPage* ixs, const SegPage* sps, const PageDev* pages,
                                                  OpenBufs bufs, const uint32_t* exits, uint32_t* entry, uint32_t* seq,
                                                  const uint32_t* flag, const uint32_t* err) {
  constexpr uint32_t NG = 8, GS = 8;  // groups of segments
  constexpr uint32_t OUT = 0xff;      // not a candidate of the next segment's first 64 bytes
  __shared__ uint32_t s_ex[64][64];
  __shared__ uint8_t s_next[64][64], s_grp[NG][64], s_ent[NG];
  __shared__ uint32_t s_pos;
  const SegPage sp = sps[blockIdx.x];
  for (uint32_t j = threadIdx.x; j < sp.nseg; j += 256) entry[sp.seg0 + j] = ~0u;
  if (threadIdx.x == 0) seq[blockIdx.x] = 0;
  if (*(const volatile uint32_t*)err != 0 || flag[sp.ix]) return;
  const PageDev& pg = pages[ixs[sp.ix].page];
  if (seg_need<F>(pg) == 0) return;
  const ChainSrc st = seg_src<F>(pg, bufs);
  const uint32_t iend = st.m + st.len;
  uint32_t pos = st.m;
  for (uint32_t b = 0; b < sp.nseg; b += 64) {
    __syncthreads();
    uint32_t ex[64 * 64 / 256];
#pragma unroll
    for (uint32_t k = 0; k < 64 * 64 / 256; ++k) {
      const uint32_t i = threadIdx.x + 256 * k;
      ex[k] = b + i / 64 < sp.nseg ? exits[(size_t)(sp.seg0 + b + i / 64) * SEG_CAND + i % 64] : ~0u;
    }
#pragma unroll
    for (uint32_t k = 0; k < 64 * 64 / 256; ++k) {
      const uint32_t i = threadIdx.x + 256 * k, c = ex[k] - SEG_BYTES;
      s_ex[i / 64][i % 64] = ex[k];
      s_next[i / 64][i % 64] = (uint8_t)(ex[k] >= SEG_BYTES && c < 64 ? c : OUT);
    }
    if (threadIdx.x == 0) s_pos = pos;
    __syncthreads();
#pragma unroll
    for (uint32_t h = 0; h < NG * 64 / 256; ++h) {
      const uint32_t i = threadIdx.x + 256 * h;
      uint32_t x = i % 64;
#pragma unroll
      for (uint32_t k = 0; k < GS; ++k) x = x == OUT ? OUT : s_next[i / 64 * GS + k][x];
      s_grp[i / 64][i % 64] = (uint8_t)x;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      const uint32_t c = pos - b * SEG_BYTES;  // (pos is not before segment b)
      uint32_t x = c < 64 && pos < iend ? c : OUT;
#pragma unroll
      for (uint32_t g = 0; g < NG; ++g) {
        s_ent[g] = (uint8_t)x;
        x = x == OUT ? OUT : s_grp[g][x];
      }
    }
    __syncthreads();
    if (threadIdx.x < NG) {
      const uint32_t g = threadIdx.x;
      uint32_t x = s_ent[g];
      if (x != OUT) {
        for (uint32_t k = 0; k < GS; ++k) {
          const uint32_t j = b + g * GS + k, q = j * SEG_BYTES + x;
          x = q < iend ? s_next[g * GS + k][x] : OUT;
          if (q < iend) entry[sp.seg0 + j] = q;
          if (x == OUT) {  // (in one group at most: the entries of those after it are OUT)
            s_pos = q;
            break;
          }
          if (g * GS + k == 63) s_pos = (j + 1) * SEG_BYTES + x;
        }
      }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      uint32_t q = s_pos;
      while (q < iend && q / SEG_BYTES < b + 64) {
        const uint32_t j = q / SEG_BYTES, c = q % SEG_BYTES;
        if (c >= seg_cands<F>()) { seq[blockIdx.x] = 1; q = ~0u; break; }
        entry[sp.seg0 + j] = q;
        const uint32_t x = c < 64 ? s_ex[j - b][c] : exits[(size_t)(sp.seg0 + j) * SEG_CAND + c];
        if (x == ~0u) { q = ~0u; break; }  // (the fill finds how many values come before)
        q = j * SEG_BYTES + x;
      }
      s_pos = q;
    }
    __syncthreads();
    pos = s_pos;
    if (pos == ~0u) break;
  }
}

// at, ent: the pieces of page ix from v0 on (SEG_DI), or of segment sg of the group
// from sg SEG_NT on.
template <int F>
__global__ __launch_bounds__(SEG_NT) void k_seg_fill(const IxPage* ixs, const SegPage* sps, const uint32_t* seg_sp,
                                                     PageDev* pages, const ChunkDev* chunks, OpenBufs bufs,
                                                     const uint32_t* entry, const uint32_t* seq, uint32_t* at,
                                                     uint8_t* ent, uint32_t* total, const uint32_t* flag,
                                                     const uint32_t* err) {
  __shared__ SegLds L;
  __shared__ uint64_t s_sum[SEG_NT / 64];
  __shared__ uint32_t s_max;
  const uint32_t sg = blockIdx.x, tid = threadIdx.x;
  const SegPage sp = sps[seg_sp[sg]];
  if (*(const volatile uint32_t*)err != 0 || flag[sp.ix] || seq[seg_sp[sg]]) return;
  const IxPage ix = ixs[sp.ix];
  PageDev& pg = pages[ix.page];
  if (F == SEG_STR && tid == 0) s_max = 0;
  const uint32_t ip = entry[sg];
  uint64_t tot = 0, before = 0, cnt = 0;
  uint32_t maxlen = 0, pe = CH_NONE;
  if (ip != ~0u) {  // (the same in every thread)
    const ChainSrc st = seg_src<F>(pg, bufs);
    const uint32_t S = (sg - sp.seg0) * SEG_BYTES, iend = st.m + st.len;
    const SegStep<F> step(&L, pg, chunks);
    uint32_t code;
    L.find(step, st.base, st.lim, S, ip, iend, code);
    const uint32_t plen = L.piece_len(S, iend), y0 = tid * CH_PIECE;
    pe = L.pent[tid];
    for (uint32_t y = pe; y < plen;) {
      uint32_t lo, hi;
      L.bytes8(y0 + y, lo, hi);
      const uint32_t a = step(lo, hi, iend - S - y0 - y, y0 + y);
      if (F == SEG_DL) ++cnt;  // (the last block need not be a full one)
      if (a == STEP_BAD || a == STEP_ODD) break;
      if (F == SEG_STR) {
        maxlen = max(maxlen, lo);
        ++cnt;
      }
      if (F == SEG_DI) cnt += hrun(lo, hi, iend - S - y0 - y, step.w).n;
      y += a;
    }
    before = wg_scan64<SEG_NT>(cnt, s_sum, tot);
  }
  const size_t pc = F == SEG_DI ? (size_t)ix.v0 + (size_t)(sg - sp.seg0) * SEG_NT + tid : (size_t)sg * SEG_NT + tid;
  if (F != SEG_DI || (sg - sp.seg0) * SEG_NT + tid < ix.nv) {
    at[pc] = sat32(before);
    ent[pc] = (uint8_t)pe;
  }
  if (tid == 0) total[sg] = sat32(tot);
  if (F == SEG_STR && pg.kind == PAGE_DICT) {
    // the dictionary's longest entry (at least: bytes after the last one may
    // make it larger, which costs the dictionary its slots at most)
    __syncthreads();
    if (maxlen) atomicMax(&s_max, maxlen);
    __syncthreads();
    if (tid == 0) atomicMax(&pg.dict_maxlen, s_max);
  }
}

// total[] becomes the values (blocks) before every segment (one wave per page).
template <int F>
__global__ __launch_bounds__(64) void k_seg_base(const IxPage* ixs, const SegPage* sps, const PageDev* pages,
                                                 uint32_t* total, const uint32_t* seq, uint32_t* flag,
                                                 const uint32_t* err) {
  const SegPage sp = sps[blockIdx.x];
  if (*(const volatile uint32_t*)err != 0 || flag[sp.ix] || seq[blockIdx.x]) return;
  uint64_t k = 0;
  for (uint32_t b = 0; b < sp.nseg; b += 64) {
    const uint32_t j = b + threadIdx.x;
    const uint64_t v = j < sp.nseg ? total[sp.seg0 + j] : 0u;
    const uint64_t incl = wave_incl_scan_u64(v);
    if (j < sp.nseg) total[sp.seg0 + j] = sat32(k + incl - v);
    k += (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)incl, 63) |
         ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(incl >> 32), 63) << 32);
  }
  if (threadIdx.x == 0 && k < seg_need<F>(pages[ixs[sp.ix].page])) flag[sp.ix] = 1;
}

__global__ __launch_bounds__(256) void k_str_ck(const IxPage* ixs, const SegPage* sps, const uint32_t* seg_sp,
                                                const PageDev* pages, OpenBufs bufs, const uint32_t* base,
                                                const uint32_t* at, const uint8_t* ent, const uint32_t* seq,
                                                uint32_t* strck, const uint32_t* flag, const uint32_t* err) {
  const uint32_t sg = blockIdx.x / (SEG_NT / 256), pc = blockIdx.x % (SEG_NT / 256) * 256 + threadIdx.x;
  const SegPage sp = sps[seg_sp[sg]];
  if (*(const volatile uint32_t*)err != 0 || flag[sp.ix] || seq[seg_sp[sg]]) return;
  const uint32_t y = ent[(size_t)sg * SEG_NT + pc];
  if (y == CH_NONE) return;
  const PageDev& pg = pages[ixs[sp.ix].page];
  const ChainSrc st = value_src(pg, bufs, 0);
  const uint32_t n = str_count(pg), iend = st.m + st.len;
  uint32_t k = base[sg] + at[(size_t)sg * SEG_NT + pc];
  uint32_t q = (sg - sp.seg0) * SEG_BYTES + pc * CH_PIECE + y;
  const uint32_t qe = min(q - y + CH_PIECE, iend);
  // the piece's value at a checkpoint, if it has one (eight values at most)
  if (k % STR_CK != 0 && k % STR_CK + 8 < STR_CK) return;
  for (; q < qe && k < n; ++k) {
    if (iend - q < 4) return;
    const uint32_t a = str_step(ld_u32(st.base, q), iend - q);
    if (a == STEP_BAD) return;
    if (k % STR_CK == 0) {
      strck[pg.strck_begin + k / STR_CK] = q - st.m;
      return;
    }
    q += a;
  }
}

__global__ __launch_bounds__(256) void k_dl_ck(const IxPage* ixs, const SegPage* sps, const uint32_t* seg_sp,
                                               PageDev* pages, const ChunkDev* chunks, OpenBufs bufs,
                                               const uint32_t* base, const uint32_t* at, const uint8_t* ent,
                                               const uint32_t* seq, uint32_t* blkpos, uint32_t* flag,
                                               const uint32_t* err) {
  const uint32_t sg = blockIdx.x / (SEG_NT / 256), pc = blockIdx.x % (SEG_NT / 256) * 256 + threadIdx.x;
  const SegPage sp = sps[seg_sp[sg]];
  if (*(const volatile uint32_t*)err != 0 || flag[sp.ix] || seq[seg_sp[sg]]) return;
  uint32_t y = ent[(size_t)sg * SEG_NT + pc];
  if (y == CH_NONE) return;
  const IxPage ix = ixs[sp.ix];
  PageDev& pg = pages[ix.page];
  const ChainSrc st = seg_src<SEG_DL>(pg, bufs);
  const uint32_t nblocks = dl_nblocks(pg), iend = st.m + st.len;
  // the stream's bytes as the blocks' step reads them
  struct Bytes {
    const ChainSrc* st;
    __device__ __forceinline__ uint32_t byte(uint32_t q) const { return q < st->m + st->len ? (uint32_t)st->base[q] : 0u; }
  } by{&st};
  const DlBlocks<Bytes> step{&by, pg.enc_m, pg.enc_w / pg.enc_m, chunks[pg.chunk].type == T_INT64 ? 64u : 32u};
  uint32_t q = (sg - sp.seg0) * SEG_BYTES + pc * CH_PIECE + y;
  const uint32_t qe = min(q - y + CH_PIECE, iend);
  for (uint32_t b = base[sg] + at[(size_t)sg * SEG_NT + pc]; q < qe && b < nblocks; ++b) {
    blkpos[ix.v0 + b] = pg.blocks_at + q - st.m;
    const uint32_t lo = ld_u32(st.base, q), hi = ld_u32(st.base, (uint64_t)q + 4);
    const bool last = b + 1 == nblocks;
    const uint32_t a = step.len(lo, hi, iend - q, q, last ? dl_used(pg, b) : pg.enc_m);
    if (a == STEP_BAD) {
      flag[sp.ix] = 1;  // (the last block, or a stream that ends early)
      return;
    }
    if (last) pg.chars_at = pg.blocks_at + q - st.m + a;
    q += a;
  }
}

// ---------------------------------------------------------------------------
// k_value_tiles: 16 lanes per tile: its values and its entry in the value
// stream, with a dictionary-index checkpoint (of every 64th value) or a block
// checkpoint per lane.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(64) void k_value_tiles(const IxPage* ixs, uint32_t nix, uint32_t tile0, uint32_t ntiles,
                                                    const PageDev* pages, const ChunkDev* chunks, OpenBufs bufs,
                                                    const uint32_t* at, const uint8_t* ent, const uint32_t* blkpos,
                                                    const uint32_t* strck, const SegPage* sps, const uint32_t* base,
                                                    const uint32_t* seq, const uint32_t* flag, TileDev* tiles, Ck* ckv,
                                                    const uint32_t* err) {
  static_assert(NSUB == 16, "16 lanes per tile");
  __shared__ uint32_t s_row[64][ROW_DW];
  if (*(const volatile uint32_t*)err != 0) return;
  const uint32_t i = blockIdx.x * 4 + threadIdx.x / 16, sub = threadIdx.x % 16;
  if (i >= ntiles) return;
  const uint32_t T = tile0 + i;
  const uint32_t ixi = ix_of_tile(ixs, nix, T);
  const IxPage ix = ixs[ixi];
  if (flag[ixi] || T - ix.tile0 >= ix.ntiles) return;
  const PageDev& pg = pages[ix.page];
  const uint32_t k0 = tiles[T].k0, k1 = T - ix.tile0 + 1 < ix.ntiles ? tiles[T + 1].k0 : pg.nonnull, nn = k1 - k0;
  const int enc = pg.encoding;
  const bool str = chunks[pg.chunk].type == T_BYTE_ARRAY;
  if (sub == 0) tiles[T].nn = nn;
  if (enc == E_PLAIN_DICT || enc == E_RLE_DICT) {
    if (sub * SUB_ROWS >= nn) return;
    const ChainSrc st = value_src(pg, bufs, 1);
    const uint32_t v = k0 + sub * SUB_ROWS, w = pg.enc_w;
    uint32_t pc, before = 0;
    if (ix.sp != ~0u && !seq[ix.sp]) {  // counts within the segment
      const SegPage sp = sps[ix.sp];
      const uint32_t j = piece_of(base + sp.base0, sp.nseg, v);
      before = base[sp.base0 + j];
      pc = j * SEG_NT;
      pc += piece_of(at + ix.v0 + pc, min(SEG_NT, ix.nv - pc), v - before);
    } else {
      pc = piece_of(at + ix.v0, ix.nv, v);
    }
    uint32_t* rowp = &s_row[threadIdx.x][0];
    row_load(rowp, st, pc);
    bool found;
    RunCur c = row_run(rowp, st, pc, ent[ix.v0 + pc], (uint64_t)before + at[ix.v0 + pc], v, w, found);
    if (!found) return;  // (not for a chain that was followed to its last value)
    c.hp += 1; c.pay += 1; c.next += 1;  // the width byte
    const uint32_t entry = (uint32_t)__builtin_amdgcn_ds_bpermute(4 * (int)(threadIdx.x & ~15u), (int)(uint32_t)c.hp);
    if (sub == 0) {
      tiles[T].val_pos = entry;
      tiles[T].val_skip = k0 - (uint32_t)c.start;
    }
    ckv[(size_t)T * NSUB + sub] = make_ck(c, (int64_t)v, w, entry);
  } else if (enc == E_DELTA || (enc == E_DLBA && str)) {
    const uint64_t B = pg.enc_w;
    if (nn == 0 || (uint64_t)k0 + nn <= 1) {  // needs no block
      if (sub == 0) tiles[T].val_pos = pg.blocks_at;
      return;
    }
    // the block holding the tile's first delta is its entry; the blocks from
    // there to the one of its last delta are its checkpoints
    const uint64_t first = k0 == 0 ? 1 : k0;
    const uint64_t bu = (first - 1) / B, lastb = ((uint64_t)k0 + nn - 2) / B;
    const uint32_t vp = blkpos[ix.v0 + bu];
    if (sub == 0) {
      tiles[T].val_pos = vp;
      tiles[T].val_skip = (uint32_t)((first - 1) % B);
    }
    if (bu + sub <= lastb) ckv[(size_t)T * NSUB + sub] = ck_at((uint64_t)(blkpos[ix.v0 + bu + sub] - vp));
  } else if (str && (enc == E_PLAIN || enc == E_DBA)) {
    // where the tile's first value starts (lane 0) and its last one ends
    if (sub > 1) return;
    const ChainSrc st = value_src(pg, bufs, 0);
    const uint32_t k = sub ? k1 : k0;
    uint32_t q = 0;
    if (k) {
      const uint32_t c = (k - 1) / STR_CK;
      q = strck[pg.strck_begin + c];
      for (uint32_t j = c * STR_CK; j < k; ++j) q += 4 + ld_u32(st.base, st.m + q);
    }
    if (sub) tiles[T].val_skip = q;
    else tiles[T].val_pos = q;
  }
}

#define CHAIN_KERNELS(NT)                                                                                             \
  template __global__ void k_levels<NT>(const IxPage*, const uint32_t*, PageDev*, OpenBufs, uint32_t*, uint32_t*,     \
                                        uint8_t*, uint32_t*, const uint32_t*);                                        \
  template __global__ void k_strings<NT>(const IxPage*, const uint32_t*, PageDev*, OpenBufs, uint32_t*, uint32_t*,    \
                                         const uint32_t*, const uint32_t*);                                           \
  template __global__ void k_di<NT>(const IxPage*, const uint32_t*, const PageDev*, OpenBufs, uint32_t*, uint8_t*,    \
                                    uint32_t*, const uint32_t*, const uint32_t*);                                     \
  template __global__ void k_dl<NT>(const IxPage*, const uint32_t*, PageDev*, const ChunkDev*, OpenBufs, uint32_t*,   \
                                    uint32_t*, const uint32_t*, const uint32_t*);
CHAIN_KERNELS(256)
CHAIN_KERNELS(1024)
#undef CHAIN_KERNELS
#define SEG_KERNELS(F)                                                                                                \
  template __global__ void k_seg_cand<F>(const IxPage*, const SegPage*, const uint32_t*, const PageDev*,              \
                                         const ChunkDev*, OpenBufs, uint32_t*, const uint32_t*, const uint32_t*);     \
  template __global__ void k_seg_link<F>(const IxPage*, const SegPage*, const PageDev*, OpenBufs, const uint32_t*,    \
                                         uint32_t*, uint32_t*, const uint32_t*, const uint32_t*);                     \
  template __global__ void k_seg_fill<F>(const IxPage*, const SegPage*, const uint32_t*, PageDev*, const ChunkDev*,   \
                                         OpenBufs, const uint32_t*, const uint32_t*, uint32_t*, uint8_t*, uint32_t*,  \
                                         const uint32_t*, const uint32_t*);                                           \
  template __global__ void k_seg_base<F>(const IxPage*, const SegPage*, const PageDev*, uint32_t*, const uint32_t*,   \
                                         uint32_t*, const uint32_t*);
SEG_KERNELS(SEG_STR)
SEG_KERNELS(SEG_DI)
SEG_KERNELS(SEG_DL)
#undef SEG_KERNELS

}  // namespace pqk
