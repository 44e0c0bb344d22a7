// pq_dba_kernels.hip -- DELTA_BYTE_ARRAY string pages (Sec. 3, Encoding
// Flexibility) expanded to the PLAIN layout, which the index pass and the
// string kernels then read as a PLAIN page's.
//
// Value k is the first prefix[k] bytes of value k - 1 followed by suffix k.
// Byte i of value k therefore comes from the suffix of the last value j <= k
// with prefix[j] <= i, so 64 values are expanded at once, one per lane,
// without waiting for each other: a lane follows its value's chain of shorter
// prefixes (the nearest earlier value with a shorter one, and so on) and
// copies each piece from the suffix it comes from; only bytes older than the
// group come from the value before it, kept in LDS.  Longer values are few to a
// group's buffer; all lanes copy them one after the other.
#include <hip/hip_runtime.h>

#include "pq_device.hpp"
#include "pq_internal.h"

namespace pqk {

constexpr uint32_t DBA_PREV = 16384;  // longest value (a page with a longer one: PQ_EUNSUPPORTED when scanned)
constexpr uint32_t DBA_SEQ = 1024;    // LDS window over a length stream
// Stretches of a group with a value longer than this: all lanes copy one value at a
// time (a lane per value idles 64 less the few that fit the buffer).  A scan of 60 MB
// of values, a lane per value / all lanes: up to 100 bytes 265 / 303 us, 150 380 / 352
// (of shared prefixes 361 / 374), 200 540 / 442, 600 2,190 / 750, 4,000 10,050 / 896.
constexpr uint32_t DBA_WHOLE = 160;

typedef uint32_t u32x4d __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) u32x4d lds_u32x4d;
typedef const __attribute__((address_space(1))) u32x4d glb_u32x4d;

__device__ __forceinline__ uint32_t first_lane(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }
// Wave-uniform byte read.
__device__ __forceinline__ uint32_t ubyte(const uint8_t* p) { return first_lane((uint32_t)*p); }

// A DELTA_BINARY_PACKED stream of 32-bit values read in order through a
// window in LDS, every field wave-uniform.
struct DeltaSeq {
  const uint8_t* s;  // stream start
  uint32_t end;      // stream bytes
  uint32_t q;        // next byte after the blocks read so far
  uint32_t B, per, M, total, done, blocks;
  uint32_t last, mind;
  uint32_t mb, used_mb, in_mb, mbq, wq, w;
  bool bad, unsupported;
  lds_u32* win;
  int32_t wlo;  // window byte i is stream byte wlo + i

  // stream bytes [a, a + n) in the window (n <= DBA_SEQ - 16; chunks past the
  // stream's last byte are not read: a chunk holding it reads at most 15 bytes
  // past it, inside the page's padding or the bytes that follow it in the file)
  __device__ void need(uint32_t a, uint32_t n) {
    if ((int32_t)a >= wlo && (int32_t)(a + n) <= wlo + (int32_t)DBA_SEQ) return;
    const uintptr_t g = (uintptr_t)(s + a) & ~(uintptr_t)15;
    wlo = (int32_t)a - (int32_t)((uintptr_t)(s + a) & 15);
    const uint32_t lane = threadIdx.x & 63;
    u32x4d v = {0u, 0u, 0u, 0u};
    if (g + 16 * lane < (uintptr_t)(s + end)) v = *(glb_u32x4d*)(g + 16 * lane);
    wave_sync();
    *(lds_u32x4d*)(win + 4 * lane) = v;
    wave_sync();
  }
  __device__ uint32_t byte(uint32_t a) {
    need(a, 1);
    return first_lane(((const lds_u8*)win)[(int32_t)a - wlo]);
  }
  __device__ uint64_t uleb() {
    uint64_t v = 0;
    for (uint32_t sh = 0;; sh += 7) {
      if (q >= end || sh > 63) { bad = true; return 0; }
      const uint32_t b = byte(q++);
      v |= (uint64_t)(b & 0x7f) << sh;
      if (!(b & 0x80)) return v;
    }
  }
  __device__ void open(const uint8_t* stream, uint32_t len, lds_u32* window) {
    s = stream; end = len; q = 0; bad = false; unsupported = false;
    win = window;
    wlo = -(int32_t)DBA_SEQ - 16;  // nothing staged
    done = 0; blocks = 0; mb = used_mb = 0; in_mb = 0; w = 0; last = 0; mind = 0; total = 0; per = 1; B = M = 1;
    mbq = wq = 0;
  }
  __device__ void init(const uint8_t* stream, uint32_t len, lds_u32* window) {
    open(stream, len, window);
    const uint64_t b = uleb(), m = uleb(), t = uleb(), f = uleb();
    if (bad || b == 0 || b % 128 != 0 || m == 0 || b % m != 0 || (b / m) % 32 != 0 || t > 0x7fffffffull) { bad = true; return; }
    if (m > 16 || b > 65536) { unsupported = true; bad = true; return; }
    B = (uint32_t)b; M = (uint32_t)m; per = B / M; total = (uint32_t)t;
    last = (uint32_t)(f >> 1) ^ (0u - (uint32_t)(f & 1));  // zigzag, 32-bit
    mbq = q; wq = q;
  }
  __device__ void block_use() {
    const uint32_t left = total - 1 - (blocks - 1) * B;
    const uint32_t used = left < B ? left : B;
    used_mb = (used + per - 1) / per;
  }
  __device__ void start_mb() {
    w = byte(wq + mb);
    if (w > 32 || (uint64_t)mbq + (uint64_t)per * w / 8 > end) bad = true;
  }
  __device__ void next_block() {
    const uint64_t md = uleb();
    mind = (uint32_t)(md >> 1) ^ (0u - (uint32_t)(md & 1));
    if (bad || M > end - q) { bad = true; return; }
    wq = q;
    q += M;
    ++blocks;
    block_use();
    mb = 0; in_mb = 0; mbq = q;
    start_mb();
  }
  // Continues at a unit's saved state, before value first.
  __device__ void resume(const uint8_t* stream, uint32_t len, lds_u32* window, const DbaStream& st, uint32_t count,
                         uint32_t first) {
    open(stream, len, window);
    q = st.q; mbq = st.mbq; wq = st.wq; last = st.last; mind = st.mind; blocks = st.blocks;
    mb = st.at >> 20; in_mb = st.at & 0xfffffu;
    B = st.B; M = st.M; per = B / M;
    total = count; done = first;
    if (q > end || mbq > end || wq > end || M > 16) { bad = true; return; }
    if (blocks) {
      block_use();
      if (mb < used_mb && mb >= end - wq) bad = true;
      else if (mb < used_mb) start_mb();
    }
  }
  __device__ DbaStream state() const {
    DbaStream st;
    st.q = q; st.mbq = mbq; st.wq = wq; st.last = last; st.mind = mind; st.blocks = blocks;
    st.at = mb << 20 | in_mb;
    st.B = B; st.M = M;
    return st;
  }
  // the next n (<= 64, <= total - done) values into buf[0, n)
  __device__ void fill(lds_u32* buf, uint32_t n, uint32_t lane) {
    uint32_t o = 0;
    if (done == 0 && n) {
      if (lane == 0) buf[0] = last;
      o = 1;
      done = 1;
    }
    while (o < n && !bad) {
      if (mb >= used_mb) { next_block(); if (bad) break; }
      const uint32_t cnt = min(n - o, per - in_mb);
      uint32_t d = 0;
      if (w) {
        const uint32_t b0 = mbq + (uint32_t)(((uint64_t)in_mb * w) >> 3);
        need(b0, (cnt * w + 7) / 8 + 9);
        if (lane < cnt) {
          const uint64_t bit = (uint64_t)(in_mb + lane) * w;
          const uint32_t a = (uint32_t)((int32_t)(mbq + (uint32_t)(bit >> 3)) - wlo);
          const uint32_t sh = (a & 3) * 8 + (uint32_t)(bit & 7);
          const uint64_t x = (((uint64_t)win[(a >> 2) + 1] << 32) | win[a >> 2]) >> sh;
          d = w == 32 ? (uint32_t)x : (uint32_t)x & ((1u << w) - 1u);
        }
      }
      const uint32_t incl = wave_incl_scan_u32(lane < cnt ? mind + d : 0u);
      const uint32_t v = last + incl;
      if (lane < cnt) buf[o + lane] = v;
      last = (uint32_t)__builtin_amdgcn_readlane((int)v, (int)(cnt - 1));
      o += cnt; done += cnt; in_mb += cnt;
      if (in_mb == per) {
        mbq += per * w / 8;
        ++mb;
        in_mb = 0;
        if (mb < used_mb) start_mb();
        else q = mbq;
      }
    }
  }
};

// One lane copies n bytes of LDS from byte a of src32 to dst.
__device__ __forceinline__ void lane_lds_copy(lds_u8* dst, const lds_u32* src32, uint32_t a, uint32_t n) {
  for (uint32_t i = 0; i < n; i += 8) {
    const uint32_t j = (a + i) >> 2, f = a & 3;
    const uint32_t d0 = src32[j], d1 = src32[j + 1], d2 = src32[j + 2];
    const uint32_t lo = __builtin_amdgcn_alignbyte(d1, d0, f), hi = __builtin_amdgcn_alignbyte(d2, d1, f);
    const uint32_t left = n - i;
#pragma unroll
    for (uint32_t k = 0; k < 8; ++k)
      if (k < left) dst[i + k] = (uint8_t)((k < 4 ? lo : hi) >> (8 * (k & 3)));
  }
}

// All lanes copy n bytes of LDS from byte a of src to byte d of dst (no overlap),
// four dwords each in flight (reads run up to 4 bytes past the source).
__device__ __forceinline__ void wave_lds_copy(lds_u32* dst, uint32_t d, const lds_u32* src, uint32_t a, uint32_t n) {
  const uint32_t lane = threadIdx.x & 63, h = min((4u - (d & 3u)) & 3u, n);
  lds_u8* db = (lds_u8*)dst;
  const lds_u8* sb = (const lds_u8*)src;
  if (lane < h) db[d + lane] = sb[a + lane];
  d += h;
  a += h;
  n -= h;
  const uint32_t m = n >> 2, q = d >> 2, j = a >> 2, f = a & 3u;
  for (uint32_t k = lane; k < m; k += 256) {
    uint32_t lo[4], hi[4];
#pragma unroll
    for (uint32_t u = 0; u < 4; ++u) {
      const uint32_t i = j + min(k + 64 * u, m - 1);
      lo[u] = src[i];
      hi[u] = src[i + 1];
    }
#pragma unroll
    for (uint32_t u = 0; u < 4; ++u)
      if (k + 64 * u < m) dst[q + k + 64 * u] = __builtin_amdgcn_alignbyte(hi[u], lo[u], f);
  }
  if (lane < (n & 3u)) db[d + 4 * m + lane] = sb[a + 4 * m + lane];
}

// ---------------------------------------------------------------------------
// k_dba, one wave per page (modes 0, 1: open) or per unit (mode 2: scans):
//   mode 0 finds the page's value stream (as the index pass does) and the
//     start of its second stream and of the suffix bytes, checks every
//     prefix against the previous value's length and the value count against
//     the page's rows, and stores the page's facts in px_out (x_src, x_len,
//     x_sfx, x_chars, xlen, x_total, x_scratch, x_ctx);
//   mode 1 expands a page from its start and records its units;
//   mode 2 expands one unit from its record: k_dba<true> the units of pages
//     whose values are at most DBA_SMALL bytes (8 KiB of LDS: 16 waves per
//     CU), k_dba<false> the others (27 KiB, five waves).
// At open the decompression layout and the expansion region are passed
// directly (open_scratch, open_out); in a scan they lie in the workspace.
// What bounds it: the dependent LDS and stream reads of a group of 64 values,
// so waves in flight: units of 256 values.  Measured on 1.35M strings of 0-40
// bytes in 256 KiB pages, a scan's expansion: 0.103 ms; 0.323 ms with units of
// 1024 values and 27 KiB of LDS per wave for all; 4.74 ms with one wave per
// page and one value at a time.
// ---------------------------------------------------------------------------
template <bool SMALL>
__global__ __launch_bounds__(64, SMALL ? 4 : 2) void k_dba(const ColScan* cols, SegTable seg, uint8_t* ws, const uint8_t* open_scratch,
                                            uint8_t* open_out, PageX* px_out, DbaUnit* units_out, int mode,
                                            uint32_t* err) {
  constexpr uint32_t PREV = SMALL ? DBA_SMALL : DBA_PREV;  // longest value
  constexpr uint32_t OUT = SMALL ? 2048 : 4096;            // a group's expanded bytes in LDS
  __shared__ uint32_t s_p[64], s_s[64], s_so[64];
  __shared__ uint8_t s_par[64];
  __shared__ __align__(16) uint32_t s_seq[2][DBA_SEQ / 4 + 4];
  __shared__ __align__(16) uint32_t s_prev[PREV / 4 + 4];
  __shared__ __align__(16) uint32_t s_win[OUT / 4 + 12];  // suffix bytes of a group
  __shared__ __align__(16) uint32_t s_out[OUT / 4 + 8];
  const uint32_t lane = threadIdx.x & 63;
  const Segment sg = seg_lookup(seg, blockIdx.x);
  uint32_t p = sg.t0 + (blockIdx.x - sg.wg0);
  if (p >= sg.t1) return;
  const ColScan* csp = cols + sg.cs;
  const FileDev fd = csp->fd;
  const DbaUnit* unit = nullptr;
  if (mode == 2) {
    unit = csp->dbau + p;
    p = unit->page;
    if (p == ~0u) return;
  }
  const PageDev pg = fd.pages[p];
  if (pg.kind == PAGE_DICT || pg.encoding != E_DBA || csp->type != T_BYTE_ARRAY) return;
  const PageX px = csp->pagex[p];
  if (mode == 2 && (px.x_maxlen <= DBA_SMALL) != SMALL) return;
  // the decompression layout (file-wide offsets)
  const uint8_t* sbase = open_scratch ? open_scratch : ws + csp->ws_scratch - csp->scratch_base;
  lds_u32* bp = (lds_u32*)&s_p[0];
  lds_u32* bs = (lds_u32*)&s_s[0];
  lds_u32* wp = (lds_u32*)&s_seq[0][0];
  lds_u32* wsq = (lds_u32*)&s_seq[1][0];
  if (!SMALL && mode == 0) {
    // the value stream, as the index pass finds it
    const bool in_scratch = pg.scratch_len > 0;
    uint64_t vo = 0, vl = 0;
    bool bad = false;
    const uint8_t* base = in_scratch ? sbase : fd.file;
    if (pg.kind == PAGE_DATA) {
      const uint64_t off = in_scratch ? pg.scratch_off : pg.payload, blen = pg.uncomp_size;
      if (csp->optional) {
        if (blen < 4) bad = true;
        else {
          const uint64_t L = ubyte(base + off) | ubyte(base + off + 1) << 8 | ubyte(base + off + 2) << 16 |
                             (uint64_t)ubyte(base + off + 3) << 24;
          if (L > blen - 4) bad = true;
          vo = off + 4 + L;
          vl = blen - 4 - L;
        }
      } else {
        vo = off;
        vl = blen;
      }
    } else if (in_scratch) {
      vo = pg.scratch_off;
      vl = pg.scratch_len;
    } else {
      const uint64_t lv = (uint64_t)pg.def_len;
      vo = pg.payload + lv;
      vl = lv <= pg.comp_size ? pg.comp_size - lv : 0;
    }
    if (bad || vl >= 0x7fffff00ull) { if (lane == 0) set_err(err, ERR_STRING, p); return; }
    const uint8_t* src = base + vo;
    DeltaSeq P, S;
    P.init(src, (uint32_t)vl, wp);
    // the prefix stream to its end: the suffix-length stream starts there
    while (!P.bad && P.done < P.total) P.fill(bp, min(64u, P.total - P.done), lane);
    // a stream ends after the miniblock holding its last value (padded)
    if (!P.bad && P.mb < P.used_mb) P.q = P.mbq + P.per * P.w / 8;
    const uint32_t sfx = P.q;
    S.open(src, 0, wsq);
    if (!P.bad) S.init(src + sfx, (uint32_t)vl - sfx, wsq);
    while (!P.bad && !S.bad && S.done < S.total) S.fill(bs, min(64u, S.total - S.done), lane);
    if (!S.bad && S.mb < S.used_mb) S.q = S.mbq + S.per * S.w / 8;
    const uint32_t chars = sfx + S.q;
    if (P.unsupported || S.unsupported) {  // valid, but not decoded here: reported when scanned
      if (lane == 0) px_out[p].x_total = DBA_UNSUPPORTED;
      return;
    }
    if (P.bad || S.bad || S.total != P.total) {
      if (lane == 0) set_err(err, ERR_DELTA, p);
      return;
    }
    // again side by side: every prefix within the previous value, every
    // value at most DBA_PREV bytes, the suffix bytes within the stream
    P.init(src, (uint32_t)vl, wp);
    S.init(src + sfx, (uint32_t)vl - sfx, wsq);
    uint64_t sum = 0, sfx_sum = 0;
    uint32_t code = 0, prevlen = 0, ctx = 0, maxlen = 0;
    while (P.done < P.total && !code) {
      const uint32_t n = min(64u, P.total - P.done), at = P.done;
      P.fill(bp, n, lane);
      S.fill(bs, n, lane);
      wave_sync();
      const uint32_t pl = lane < n ? bp[lane] : 0u, sl = lane < n ? bs[lane] : 0u;
      const uint64_t L = (uint64_t)pl + sl;
      const uint32_t before = (uint32_t)__shfl_up((int)(uint32_t)L, 1);
      const bool broken = lane < n && (pl > (lane ? before : prevlen) || (int32_t)pl < 0 || (int32_t)sl < 0);
      const bool longer = lane < n && !broken && L > DBA_PREV;
      // the first value that is not decoded decides
      const uint64_t mb = __ballot(broken), ml = __ballot(longer);
      if (mb | ml) {
        code = (mb && (!ml || __builtin_ctzll(mb) < __builtin_ctzll(ml))) ? ERR_STRING : ERR_UNSUPPORTED;
        break;
      }
      maxlen = max(maxlen, (uint32_t)L);
      const uint32_t tl = wave_incl_scan_u32((uint32_t)L), ts = wave_incl_scan_u32(sl);
      sum += 4ull * n + (uint32_t)__builtin_amdgcn_readlane((int)tl, 63);
      sfx_sum += (uint32_t)__builtin_amdgcn_readlane((int)ts, 63);
      prevlen = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)L, (int)(n - 1));
      if (at % DBA_UNIT == 0) ctx += (first_lane(pl) + 15u) & ~15u;
      wave_sync();
    }
    if (!code && ((uint64_t)chars + sfx_sum > vl || sum >= 0x80000000ull)) code = ERR_STRING;
    if (code == ERR_UNSUPPORTED) { if (lane == 0) px_out[p].x_total = DBA_UNSUPPORTED; return; }
    // the units and the bytes they keep are reserved by the page's rows: a
    // stream of more values would have mode 1 write past them
    if (!code && P.total > (uint32_t)pg.num_values) code = ERR_VALUES;
    if (code) { if (lane == 0) set_err(err, code, p); return; }
    for (int m = 32; m; m >>= 1) maxlen = max(maxlen, (uint32_t)__shfl_xor((int)maxlen, m));
    if (lane == 0) {
      PageX& o = px_out[p];
      o.x_maxlen = maxlen;
      o.x_src = vo;
      o.x_len = (uint32_t)vl;
      o.x_sfx = sfx;
      o.x_chars = chars;
      o.xlen = (uint32_t)sum;
      o.x_total = P.total;
      o.x_scratch = in_scratch ? 1u : 0u;
      o.x_ctx = ctx;
    }
    return;
  }
  // modes 1 and 2: the values in the PLAIN layout
  if (px.x_total == DBA_UNSUPPORTED) return;
  const uint8_t* src = (px.x_scratch ? sbase : fd.file) + px.x_src;
  uint8_t* out = open_out ? open_out + px.x_off : ws + csp->ws_xscratch + (px.x_off - csp->xscratch_base);
  lds_u8* prev = (lds_u8*)&s_prev[0];
  DeltaSeq P, S;
  uint32_t pos = 0, c = 0, last = px.x_total, ctx = 0;
  if (!SMALL && mode == 1) {
    P.init(src, px.x_len, wp);
    S.init(src + px.x_sfx, px.x_len - px.x_sfx, wsq);
  } else {
    const DbaUnit u = *unit;
    P.resume(src, px.x_len, wp, u.p, px.x_total, u.first);
    S.resume(src + px.x_sfx, px.x_len - px.x_sfx, wsq, u.s, px.x_total, u.first);
    pos = u.pos;
    c = u.c;
    last = min(u.first + DBA_UNIT, px.x_total);
    for (uint32_t i = lane; i < min(u.ctx_len, PREV); i += 64) prev[i] = u.ctx[i];
  }
  if (P.bad || S.bad) { if (lane == 0) set_err(err, ERR_DELTA, p); return; }
  const uint8_t* chars = src + px.x_chars;
  const uint32_t nchars = px.x_len - px.x_chars;
  lds_u8* ob = (lds_u8*)&s_out[0];
  lds_u32 *ob32 = (lds_u32*)&s_out[0], *prev32 = (lds_u32*)&s_prev[0], *win32 = (lds_u32*)&s_win[0];
  // suffix bytes [at, at + m) to the window, m <= OUT; returns where the first lies
  auto load_win = [&](uint32_t at, uint32_t m) -> uint32_t {
    const uintptr_t g0 = (uintptr_t)(chars + at) & ~(uintptr_t)15;
    const uint32_t lead = (uint32_t)((uintptr_t)(chars + at) - g0);
    const uintptr_t gend = (uintptr_t)(chars + nchars);
    for (uint32_t k = lane; 16 * k < lead + m; k += 64) {
      u32x4d v = {0u, 0u, 0u, 0u};
      if (g0 + 16 * k < gend) v = *(glb_u32x4d*)(g0 + 16 * k);
      *(lds_u32x4d*)((lds_u32*)&s_win[0] + 4 * k) = v;
    }
    return lead;
  };
  // m bytes of the LDS buffer from byte head on to o (whose place in its 16 bytes is head)
  auto flush = [&](uint8_t* o, uint32_t head, uint32_t m) {
    uint8_t* g = o - head;
    const uint32_t tot = head + m;
    for (uint32_t k = 16 * lane; k < tot; k += 1024) {
      const u32x4d v = *(const lds_u32x4d*)((lds_u32*)&s_out[0] + (k >> 2));
      if (k >= head && k + 16 <= tot) {
        *(__attribute__((address_space(1))) u32x4d*)(g + k) = v;
      } else {
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (uint32_t i = 0; i < 16; ++i)
          if (k + i >= head && k + i < tot) g[k + i] = (uint8_t)(w[i >> 2] >> (8 * (i & 3)));
      }
    }
  };
  while (P.done < last) {
    const uint32_t n = min(64u, last - P.done), at = P.done;
    DbaStream ps{}, ss{};
    const bool rec = !SMALL && mode == 1 && at % DBA_UNIT == 0;
    if (rec) { ps = P.state(); ss = S.state(); }
    P.fill(bp, n, lane);
    S.fill(bs, n, lane);
    if (P.bad || S.bad) { if (lane == 0) set_err(err, ERR_DELTA, p); return; }
    wave_sync();
    const uint32_t pl = lane < n ? bp[lane] : 0u, sl = lane < n ? bs[lane] : 0u;
    if (rec) {
      const uint32_t cl = min(first_lane(pl), PREV);
      for (uint32_t i = lane; i < cl; i += 64) px.x_ctxp[ctx + i] = prev[i];
      if (lane == 0) {
        DbaUnit& u = units_out[px.x_unit0 + at / DBA_UNIT];
        u.p = ps;
        u.s = ss;
        u.ctx = px.x_ctxp + ctx;
        u.ctx_len = cl;
        u.first = at;
        u.c = c;
        u.pos = pos;
        u.page = p;
      }
      ctx += (cl + 15u) & ~15u;
    }
    if (__ballot(pl > PREV || sl > PREV || pl + sl > PREV)) { if (lane == 0) set_err(err, ERR_STRING, p); return; }
    const uint32_t L = pl + sl;
    const uint32_t si = wave_incl_scan_u32(sl), oi = wave_incl_scan_u32(lane < n ? 4 + L : 0u);
    if ((uint64_t)c + (uint32_t)__builtin_amdgcn_readlane((int)si, 63) > nchars ||
        (uint64_t)pos + (uint32_t)__builtin_amdgcn_readlane((int)oi, 63) > px.xlen) {
      if (lane == 0) set_err(err, ERR_STRING, p);
      return;
    }
    // the nearest earlier value of the group with a shorter prefix (0xff: none)
    uint32_t par = 0xffu;
    if (__ballot(pl != 0)) {
      for (uint32_t j = 0; j + 1 < n; ++j) {
        const uint32_t x = (uint32_t)__builtin_amdgcn_readlane((int)pl, (int)j);
        if (lane > j && x < pl) par = j;
      }
    }
    s_so[lane] = si - sl;
    s_par[lane] = (uint8_t)par;
    // stretches of the group's expanded bytes that fit the LDS buffer: whole
    // values [a, b), or a part of one value over the buffer
    for (uint32_t a = 0; a < n;) {
      const uint32_t o0 = a ? (uint32_t)__builtin_amdgcn_readlane((int)oi, (int)(a - 1)) : 0u;
      const uint32_t s0 = a ? (uint32_t)__builtin_amdgcn_readlane((int)si, (int)(a - 1)) : 0u;
      const uint64_t fit = __ballot(lane >= a && lane < n && oi - o0 <= OUT);
      uint32_t b = a + (uint32_t)__popcll(fit);
      if (b == a) {  // one value over the buffer
        b = a + 1;
        const uint32_t vp = (uint32_t)__builtin_amdgcn_readlane((int)pl, (int)a);
        const uint32_t vn = 4 + (uint32_t)__builtin_amdgcn_readlane((int)L, (int)a);
        for (uint32_t x0 = 0; x0 < vn; x0 += OUT) {
          const uint32_t x1 = min(vn, x0 + OUT), xs = max(x0, 4 + vp);  // its bytes; those from xs on are suffix
          uint32_t lead = 0;
          wave_sync();
          if (xs < x1) lead = load_win(c + s0 + (xs - 4 - vp), x1 - xs);
          const uint32_t head = (uint32_t)((uintptr_t)(out + pos + o0 + x0) & 15);
          wave_sync();
          const uint32_t xp = max(x0, 4u);
          if (x0 == 0 && lane < 4) ob[head + lane] = (uint8_t)((vn - 4) >> (8 * lane));
          if (xp < min(x1, 4 + vp)) wave_lds_copy(ob32, head + (xp - x0), prev32, xp - 4, min(x1, 4 + vp) - xp);
          if (xs < x1) {
            wave_lds_copy(ob32, head + (xs - x0), win32, lead, x1 - xs);
            wave_lds_copy(prev32, xs - 4, win32, lead, x1 - xs);
          }
          wave_sync();
          flush(out + pos + o0 + x0, head, x1 - x0);
        }
        wave_sync();
      } else {
        const uint32_t s1 = (uint32_t)__builtin_amdgcn_readlane((int)si, (int)(b - 1));
        const uint32_t o1 = (uint32_t)__builtin_amdgcn_readlane((int)oi, (int)(b - 1));
        wave_sync();
        const uint32_t lead = load_win(c + s0, s1 - s0);
        // the LDS buffer has the output's place in its 16 bytes
        const uint32_t head = (uint32_t)((uintptr_t)(out + pos + o0) & 15);
        wave_sync();
        if (__ballot(lane >= a && lane < b && L > DBA_WHOLE)) {
          // long values: one after the other
          uint32_t from = 0, keep = ~0u;
          for (uint32_t j = a; j < b; ++j) {
            const uint32_t vp = (uint32_t)__builtin_amdgcn_readlane((int)pl, (int)j);
            const uint32_t vl = (uint32_t)__builtin_amdgcn_readlane((int)L, (int)j);
            const uint32_t at = head + (uint32_t)__builtin_amdgcn_readlane((int)oi, (int)j) - o0 - 4 - vl;
            const uint32_t w0 = lead + (uint32_t)__builtin_amdgcn_readlane((int)(si - sl), (int)j) - s0;
            if (lane < 4) ob[at + lane] = (uint8_t)(vl >> (8 * lane));
            if (vp) wave_lds_copy(ob32, at + 4, j == a ? prev32 : ob32, j == a ? 0u : from, vp);
            if (vl > vp) wave_lds_copy(ob32, at + 4 + vp, win32, w0, vl - vp);
            wave_sync();
            from = at + 4;
            keep = min(keep, vp);
          }
          // the last one is the next stretch's predecessor; its bytes that all the
          // stretch's values share with the one before it are there
          const uint32_t vl = (uint32_t)__builtin_amdgcn_readlane((int)L, (int)(b - 1));
          if (vl > keep) wave_lds_copy(prev32, keep, ob32, from + keep, vl - keep);
        } else {
          if (lane >= a && lane < b) {
            lds_u8* d = ob + head + (oi - 4 - L - o0);
#pragma unroll
            for (uint32_t k = 0; k < 4; ++k) d[k] = (uint8_t)(L >> (8 * k));
            d += 4;
            lane_lds_copy(d + pl, (const lds_u32*)&s_win[0], lead + (si - sl - s0), sl);
            // the prefix, from its end: pieces of the values with shorter
            // prefixes, the rest from the value before the run
            uint32_t hi = pl, j = par;
            while (hi) {
              if (j == 0xffu || j < a) {
                lane_lds_copy(d, (const lds_u32*)&s_prev[0], 0, hi);
                break;
              }
              const uint32_t lo = bp[j];
              lane_lds_copy(d + lo, (const lds_u32*)&s_win[0], lead + (s_so[j] - s0), hi - lo);
              hi = lo;
              j = s_par[j];
            }
          }
          wave_sync();
          // the run's last value is the next one's predecessor
          const uint32_t vl = (uint32_t)__builtin_amdgcn_readlane((int)L, (int)(b - 1));
          for (uint32_t i = lane; i < vl; i += 64) prev[i] = ob[head + (o1 - o0) - vl + i];
        }
        flush(out + pos + o0, head, o1 - o0);
        wave_sync();
      }
      a = b;
    }
    pos += (uint32_t)__builtin_amdgcn_readlane((int)oi, 63);
    c += (uint32_t)__builtin_amdgcn_readlane((int)si, 63);
  }
}

template __global__ void k_dba<false>(const ColScan*, SegTable, uint8_t*, const uint8_t*, uint8_t*, PageX*, DbaUnit*, int,
                                      uint32_t*);
template __global__ void k_dba<true>(const ColScan*, SegTable, uint8_t*, const uint8_t*, uint8_t*, PageX*, DbaUnit*, int,
                                     uint32_t*);

}  // namespace pqk
