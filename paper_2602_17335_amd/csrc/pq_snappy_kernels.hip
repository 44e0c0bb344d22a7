// pq_snappy_kernels.hip -- Snappy pages with a block index (Sec. 2: chunk
// compression undone by GPU kernels before the decode): the index built when
// a file is opened and the block decoder of every scan.
//
// A Snappy stream is a chain of elements (a literal or a copy of earlier
// output), each found from the one before it, and a compressor of the usual
// kind cuts its input into 64 KiB blocks that share no copy.  The index
// (k_snap_index) holds where each block's elements start in the stream and
// one bit per stream byte that is set where an element starts.  With the
// bits, no thread follows the chain: k_snappy_blk parses a block's stream
// 8 KiB at a time, all threads at once, and keeps the block's output in LDS,
// so that only copies of copies wait for each other.
#include <hip/hip_runtime.h>

#include "pq_chain.hpp"
#include "pq_device.hpp"
#include "pq_internal.h"

namespace pqk {

typedef uint32_t u32x4s __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2s __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) u32x4s lds_u32x4;
typedef __attribute__((address_space(3))) uint16_t lds_u16;

// One element from its first five bytes (x: bytes 0..3, x4: byte 4).
struct SnapEl {
  uint32_t len;  // output bytes
  uint32_t hl;   // tag and length or offset bytes
  uint32_t off;  // copies: offset
  bool lit;
};
__device__ __forceinline__ SnapEl snap_el(uint32_t x, uint32_t x4) {
  const uint32_t t = x & 0xffu, ty = t & 3u, l6 = t >> 2;
  const uint32_t b1234 = (x >> 8) | (x4 << 24);
  SnapEl e;
  e.lit = ty == 0u;
  // a literal: length l6 + 1, or (l6 >= 60) the next l6 - 59 bytes + 1
  const uint32_t nbb = l6 >= 60u ? l6 - 59u : 0u;
  const uint32_t lsh = (32u - 8u * nbb) & 31u;
  const uint32_t lext = (b1234 << lsh) >> lsh;
  // a copy with a 1-byte (ty 1), 2-byte (2) or 4-byte (3) offset
  const bool c1 = ty == 1u;
  const uint32_t clen = c1 ? 4u + (l6 & 7u) : l6 + 1u;
  e.off = c1 ? ((t >> 5) << 8) | (b1234 & 0xffu) : b1234 & (ty == 2u ? 0xffffu : 0xffffffffu);
  e.len = e.lit ? (nbb ? lext : l6) + 1u : clen;
  e.hl = e.lit ? 1u + nbb : ty + 1u + (ty == 3u ? 1u : 0u);
  return e;
}

// A compressed page's stream: bytes [m, m + n) of a 16-byte aligned base,
// readable up to lim (a multiple of 16).
struct SnapSrc {
  const uint8_t* base;
  uint32_t m, n, lim;
  bool fits;  // offsets fit 31 bits
};
__device__ __forceinline__ SnapSrc snap_src(const uint8_t* file, const PageDev& pg) {
  uint64_t off = pg.payload, len = pg.comp_size;
  if (pg.kind == PAGE_DATA_V2) {
    const uint64_t lev = (uint64_t)pg.def_len;
    off += lev;
    len = len > lev ? len - lev : 0;
  }
  SnapSrc s;
  s.m = (uint32_t)(off & 15);
  s.base = file + (off - s.m);
  s.fits = len < 0x7fffffe0ull;
  s.n = s.fits ? (uint32_t)len : 0;
  s.lim = (s.m + s.n + 15u) & ~15u;
  return s;
}

// ---------------------------------------------------------------------------
// k_snap_index (open): the block index of every compressed page, one
// workgroup per page.  Entry b of a page is the stream offset of the element
// that starts output block b; the page's first entry is SBLK_NONE when an
// element straddles a block boundary, a copy reaches before the start of its
// block, or the stream is malformed: such a page is decompressed
// sequentially by k_snappy, which reports what is wrong.
//
// The chain is found in 32 KiB segments (pq_chain.hpp); every thread then
// walks its piece's elements (at most 16): lengths, the output before the piece
// that its copies need, a prefix sum over the pieces, the checks, the start bits,
// and, in a piece where a block starts, the elements again for the block starts.
// What bounds it: the dependent LDS reads of the chain's steps.  Measured on a
// 2M-row wide table with 1 MiB pages: 1.03 ms (1.08 with every piece's
// elements walked twice); one wave per page that walks the
// tags from a staged window, 51.7 ms (0.2 us per element of the densest page).
// ---------------------------------------------------------------------------
constexpr uint32_t SX_WG = 1024;

__global__ __launch_bounds__(SX_WG) void k_snap_index(const ColScan* cols, SegTable seg) {
  __shared__ ChainLds<SX_WG, 64> L;
  __shared__ uint32_t s_sum[SX_WG / 64];
  const Segment sg = seg_lookup(seg, blockIdx.x);
  const uint32_t p = sg.t0 + (blockIdx.x - sg.wg0);
  if (p >= sg.t1) return;
  const ColScan* cs = cols + sg.cs;
  const PageDev* pg = cs->fd.pages + p;
  const uint32_t total = pg->scratch_len;
  if (total == 0) return;
  const SnapSrc src = snap_src(cs->fd.file, *pg);
  uint32_t* sblk = cs->fd.sblk + pg->sblk_begin;
  uint32_t* bits = reinterpret_cast<uint32_t*>(cs->fd.sbits + 8ull * pg->sbit0);
  const uint32_t nbits = snap_bit_words(src.m, src.n);  // words of the page's start bits
  const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint32_t iend = src.m + src.n;
  bool ok = src.fits;
  uint32_t ip = src.m;
  {  // stream length (varint)
    uint64_t v = 0;
    int sft = 0;
    for (;;) {
      if (!ok || ip >= iend || sft > 28) { ok = false; break; }
      const uint32_t b = src.base[ip++];
      v |= (uint64_t)(b & 0x7f) << sft;
      if (!(b & 0x80)) break;
      sft += 7;
    }
    if (ok && v != total) ok = false;
  }
  const uint32_t first = ip - src.m;
  uint32_t op = 0, wz = 0;  // output bytes so far; start-bit words written
  auto step = [](uint32_t lo, uint32_t hi, uint32_t left, uint32_t) -> uint32_t {
    const SnapEl e = snap_el(lo, hi & 0xffu);
    if (e.hl > left || (e.lit && (e.len - 1u >= SNAP_BLOCK || e.len > left - e.hl))) return STEP_BAD;
    return e.hl + (e.lit ? e.len : 0u);
  };
  while (ok && ip < iend) {
    const uint32_t S = ip & ~(CH_PIECE - 1);
    for (uint32_t w = wz + tid; w < min(S / CH_PIECE, nbits); w += SX_WG) bits[w] = 0;
    uint32_t code;
    const uint32_t next = L.find(step, src.base, src.lim, S, ip, iend, code);
    ok = code == 0;
    if (!ok) break;
    // the piece's elements: lengths and start bits
    const uint32_t plen = L.piece_len(S, iend), y0 = tid * CH_PIECE;
    uint32_t mask = 0, sum = 0;
    uint32_t reach = 0;  // output bytes before the piece's that its copies need
    bool bad = false;
    for (uint32_t y = L.pent[tid]; y < plen;) {
      uint32_t lo, hi;
      L.bytes8(y0 + y, lo, hi);
      const SnapEl e = snap_el(lo, hi & 0xffu);
      mask |= 1u << y;
      if (!e.lit) {
        bad |= e.off == 0;
        reach = max(reach, e.off > sum ? e.off - sum : 0u);
      }
      sum += e.len;
      y += e.hl + (e.lit ? e.len : 0u);
    }
    wz = S / CH_PIECE + SX_WG;
    if (S / CH_PIECE + tid < nbits) bits[S / CH_PIECE + tid] = mask;
    const uint32_t incl = wave_incl_scan_u32(sum);
    if (lane == 63) s_sum[wave] = incl;
    __syncthreads();
    uint32_t o = op + incl - sum, tot = 0;
#pragma unroll
    for (uint32_t w = 0; w < SX_WG / 64; ++w) {
      const uint32_t v = s_sum[w];
      if (w < wave) o += v;
      tot += v;
    }
    // checks and block starts: element by element where a block starts in the piece
    const uint32_t ob0 = o & (SNAP_BLOCK - 1);
    const bool starts = ob0 == 0 || sum > SNAP_BLOCK - ob0;
    if (mask) bad |= o > total || sum > total - o || (!starts && reach > ob0);
    for (uint32_t m = starts && !bad ? mask : 0u; m; m &= m - 1) {
      const uint32_t y = (uint32_t)__builtin_ctz(m);
      uint32_t lo, hi;
      L.bytes8(y0 + y, lo, hi);
      const SnapEl e = snap_el(lo, hi & 0xffu);
      const uint32_t ob = o & (SNAP_BLOCK - 1);
      bad |= o >= total || e.len > total - o || e.len > SNAP_BLOCK - ob || (!e.lit && (e.off == 0 || e.off > ob));
      if (!bad && ob == 0 && o) sblk[o / SNAP_BLOCK] = S + y0 + y - src.m;
      o += e.len;
    }
    // (a segment's lengths sum to less than 2^30: pieces hold at most 16
    // elements, a literal's bytes count once)
    if (__syncthreads_or(bad || op > total || tot > total - op)) { ok = false; break; }
    op += tot;
    ip = next;
  }
  if (op != total || ip != iend) ok = false;
  for (uint32_t w = wz + tid; w < nbits; w += SX_WG) bits[w] = 0;
  if (tid == 0) sblk[0] = ok ? first : SBLK_NONE;
}

// ---------------------------------------------------------------------------
// k_snappy_blk: one workgroup per 64 KiB output block.  The block's output
// is built in LDS and streamed out as it becomes final.  A pass takes 8 KiB
// of the stream, 16 bytes per thread in registers:
//   - a thread decodes the elements that start in its bytes (the start bits
//     say where; at most 8), a prefix sum over the threads gives their output
//     positions, and each thread stores those of its bytes that are literal
//     data (a literal that began in an earlier thread's bytes is passed on
//     with the sum);
//   - the copies go into a list in the order of the output, one or two per
//     thread (in the threads that found them, a dense wave would run each
//     step for up to 8 copies a lane, a sparse one for a few lanes);
//   - those whose source lies before the pass's output are done at once;
//     the others mark their output bytes in a bit map of pending bytes, and,
//     after a barrier, each is done as soon as no byte of its source is
//     pending.  Waves need no further barrier for this: a wave's LDS accesses
//     are performed in order, a copy's bytes before its bits are cleared, and
//     the first pending copy never waits.
// Consecutive copies of one thread with the same offset of at most 64 (runs)
// share one source, the bytes before the first of them.  A copy whose source
// lies within the thread's last copy takes that one's source instead: in a
// column of sorted values every value copies most bytes of the value before it,
// a chain as long as the page whose every link waits for the one before (a
// sorted INT64 column of 31,000 pages of 4 KiB: 1,860 us, with the links between a
// thread's four copies taken out 763; one lane per page, element by element, 723).
// What bounds it: the rounds of copies of copies (up to 220 deep in a block
// of the wide table, a few in most) and, in blocks of literals, the LDS byte
// stores and the stream loads in flight.
// Two workgroups of 512 threads fit a CU's LDS (64 KiB output, 8 KiB bit map).
// Measured on the 4M-row wide table (5,056 blocks): 0.87 ms a scan, 7,600 vector
// instructions per wave and block (0.5 ms of issue); with the copies left to
// the threads that found them 1.73 ms; with one lane per block and the loads of
// 8 elements in flight together 10.8 ms, its densest block's 2,100 round trips,
// however few the blocks.
// ---------------------------------------------------------------------------
constexpr uint32_t SB_BYTES = 16;  // stream bytes per thread and pass
// The shape for blocks of at most OUT output bytes: threads, and copies done side by
// side (what the LDS of 2, 8 and 15 workgroups per CU leaves).
template <uint32_t OUT>
struct SbShape {
  static constexpr uint32_t WG = 512, LIST = 944;
};
// A page of a few KiB is one or two of the large shape's passes, and two such
// workgroups hold a CU.
template <>
struct SbShape<SNAP_SHAPE[1]> {
  static constexpr uint32_t WG = 128, LIST = 240;
};
// A page of up to 8 KiB: one wave, whose passes need no barrier (pages of 4 KiB that
// are one literal, 30,000 of DOUBLE values: 152 us by two waves, now 112; by one lane
// each 118).
template <>
struct SbShape<SNAP_SHAPE[0]> {
  static constexpr uint32_t WG = 64, LIST = 120;
};
constexpr int SB_EL = SB_BYTES / 2;  // elements starting in a thread's bytes (each takes two or more)

// Bits [a, a + n) of the pending map, n <= 64: whether any is set.
__device__ __forceinline__ bool pend_any(const uint32_t* pend, uint32_t a, uint32_t n) {
  const uint32_t i = a >> 5, sh = a & 31;
  const uint32_t w0 = __hip_atomic_load(pend + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  const uint32_t w1 = __hip_atomic_load(pend + i + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  const uint32_t w2 = __hip_atomic_load(pend + i + 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  uint64_t v = (((uint64_t)w1 << 32) | w0) >> sh;
  if (sh) v |= (uint64_t)w2 << (64 - sh);
  return (n >= 64 ? v : v & ((1ull << n) - 1)) != 0;
}
// Sets (or clears) bits [a, a + n) of the pending map, 1 <= n <= 64.
template <bool SET>
__device__ __forceinline__ void pend_mark(uint32_t* pend, uint32_t a, uint32_t n) {
  const uint32_t i = a >> 5, sh = a & 31;
  const uint64_t m = n >= 64 ? ~0ull : (1ull << n) - 1;
  const uint64_t lo = m << sh;
  const uint32_t w[3] = {(uint32_t)lo, (uint32_t)(lo >> 32), sh ? (uint32_t)(m >> (64 - sh)) : 0u};
#pragma unroll
  for (int k = 0; k < 3; ++k)
    if (w[k]) {
      if (SET) __hip_atomic_fetch_or(pend + i + k, w[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      else __hip_atomic_fetch_and(pend + i + k, ~w[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
}

// n <= 64 bytes of the block's output to position o: from s on (no overlap
// with the destination), or repeating with period per (per < n) from s, the
// first one byte r of the period.
__device__ __forceinline__ void snap_copy(lds_u8* out, uint32_t o, uint32_t s, uint32_t n, uint32_t per, uint32_t r) {
  if (per == 0) {
    lds_u32* out32 = (lds_u32*)out;
    for (uint32_t i = 0; i < n; i += 8) {
      const uint32_t a = s + i, j = a >> 2;
      const uint32_t d0 = out32[j], d1 = out32[j + 1], d2 = out32[j + 2];
      const uint32_t lo = __builtin_amdgcn_alignbyte(d1, d0, a & 3), hi = __builtin_amdgcn_alignbyte(d2, d1, a & 3);
      lds_u8* d = out + o + i;
      const uint32_t left = n - i;
#pragma unroll
      for (uint32_t k = 0; k < 8; ++k)
        if (k < left) d[k] = (uint8_t)((k < 4 ? lo : hi) >> (8 * (k & 3)));
    }
  } else {
    for (uint32_t i = 0; i < n; i += 8) {
      uint32_t b[8];
#pragma unroll
      for (uint32_t k = 0; k < 8; ++k) {
        b[k] = out[s + r];
        r = r + 1 == per ? 0u : r + 1;
      }
#pragma unroll
      for (uint32_t k = 0; k < 8; ++k)
        if (i + k < n) out[o + i + k] = (uint8_t)b[k];
    }
  }
}

// dicts = 1 (open): dictionary pages too.
template <uint32_t OUT>
__global__ __launch_bounds__(SbShape<OUT>::WG, 4) void k_snappy_blk(const ColScan* cols, SegTable seg, uint8_t* ws,
                                                                    uint32_t* err, int dicts) {
  constexpr uint32_t SB_WG = SbShape<OUT>::WG, SB_LIST = SbShape<OUT>::LIST, SB_PASS = SB_WG * SB_BYTES;
  static_assert(SB_LIST <= 2 * SB_WG, "a thread takes at most two copies of the list");
  __shared__ __align__(16) uint32_t s_out[OUT / 4 + 4];  // (reads run up to 10 bytes past a source)
  __shared__ uint32_t s_pend[OUT / 32 + 2];
  __shared__ u32x2s s_list[SB_LIST];
  __shared__ __align__(16) uint32_t s_x[2][SB_WG / 64][4];
  const Segment sg = seg_lookup(seg, blockIdx.x);
  const uint32_t b = sg.t0 + (blockIdx.x - sg.wg0);
  if (b >= sg.t1) return;
  const ColScan* cs = cols + sg.cs;
  const uint32_t p = cs->fd.sblk_page[b];
  const PageDev* pg = cs->fd.pages + p;
  if (pg->scratch_len == 0 || (pg->kind == PAGE_DICT && !dicts)) return;  // dictionaries: decompressed at open
  if (dicts && !open_sel_ok(*cs, *pg)) return;
  const uint32_t* sblk = cs->fd.sblk;
  const uint32_t fb = pg->sblk_begin, kb = b - fb, total = pg->scratch_len;
  if (sblk[fb] == SBLK_NONE) return;  // decoded sequentially by k_snappy
  const SnapSrc src = snap_src(cs->fd.file, *pg);
  const uint32_t nblk = (total + SNAP_BLOCK - 1) / SNAP_BLOCK;
  const uint32_t i0 = sblk[b], i1 = kb + 1 < nblk ? sblk[b + 1] : src.n;
  const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (!src.fits || i0 > i1 || i1 > src.n) {
    if (tid == 0) set_err(err, ERR_SNAPPY, p);
    return;
  }
  const uint16_t* bits = cs->fd.sbits + 8ull * pg->sbit0;
  uint8_t* dst = ws + cs->ws_scratch + (pg->scratch_off - cs->scratch_base) + (uint64_t)kb * SNAP_BLOCK;
  const uint32_t blen = min(SNAP_BLOCK, total - kb * SNAP_BLOCK);
  const uint32_t q0 = src.m + i0, qe = src.m + i1;
  lds_u8* out = (lds_u8*)&s_out[0];
  if (blen > OUT) {  // (the launch's pages are smaller)
    if (tid == 0) set_err(err, ERR_SNAPPY, p);
    return;
  }
  for (uint32_t i = tid; i < OUT / 32 + 2; i += SB_WG) s_pend[i] = 0;

  uint32_t A = q0 & ~15u;  // stream position of the pass
  u32x4s nw = {0u, 0u, 0u, 0u};
  uint32_t nw4 = 0, nmask = 0;  // the next pass's bytes and start bits
  auto fetch = [&](uint32_t q) {
    nw = u32x4s{0u, 0u, 0u, 0u};
    nw4 = 0;
    nmask = 0;
    if (q < qe) {
      nw = *reinterpret_cast<const u32x4s*>(src.base + q);
      nmask = bits[q >> 4];
    }
    if (q + 16 < src.lim) nw4 = *reinterpret_cast<const uint32_t*>(src.base + q + 16);
  };
  fetch(A + SB_BYTES * tid);
  uint32_t op = 0;               // output position of the pass's first element
  uint32_t fin = 0;              // output bytes final before the pass (fewer: a literal goes on in it)
  uint32_t cov_d = ~0u, cov_o = 0;  // the last element before it: a literal's first data byte (~0: a copy)
                                    // in the stream and its output position
  uint32_t flushed = 0;
  bool bad = false;
  for (uint32_t par = 0; A < qe; A += SB_PASS, par ^= 1) {
    const uint32_t q = A + SB_BYTES * tid;
    const uint32_t w0 = nw.x, w1 = nw.y, w2 = nw.z, w3 = nw.w, w4 = nw4;
    uint32_t mask = nmask;
    if (q < q0) mask &= ~0u << (q0 - q);
    const uint32_t inb = q < qe ? min(qe - q, SB_BYTES) : 0u;  // this thread's bytes of the block's stream
    mask &= (1u << inb) - 1u;
    if (A + SB_PASS < qe) fetch(q + SB_PASS);
    // the elements: el[j] output bytes, ei[j] offset (16 bits; 0: a literal,
    // or invalid), start byte (4 bits), header bytes (3 bits), literal flag
    uint32_t el[SB_EL], ei[SB_EL];
    uint32_t sum = 0, last_d = ~0u, last_o = 0, nc = 0;  // output bytes, the last element, copies
    {
      uint32_t mk = mask;
#pragma unroll
      for (int j = 0; j < SB_EL; ++j) {
        el[j] = 0;
        ei[j] = 0;
        if (mk) {
          const uint32_t k = (uint32_t)__builtin_ctz(mk), c = k >> 2;
          mk &= mk - 1;
          const uint32_t lo = c < 2 ? (c ? w1 : w0) : (c == 2 ? w2 : w3);
          const uint32_t hi = c < 2 ? (c ? w2 : w1) : (c == 2 ? w3 : w4);
          const uint32_t x = __builtin_amdgcn_alignbyte(hi, lo, k & 3), x4 = (hi >> (8 * (k & 3))) & 0xffu;
          const SnapEl e = snap_el(x, x4);
          const uint32_t left = qe - (q + k);
          const bool inv = e.hl > left || e.len - 1u >= SNAP_BLOCK ||
                           (e.lit ? e.len > left - e.hl : (e.off - 1u >= SNAP_BLOCK - 1u));
          bad |= inv;
          el[j] = inv ? 0u : e.len;
          ei[j] = (e.lit || inv ? 0u : e.off) | (k << 16) | (e.hl << 20) | ((e.lit && !inv ? 1u : 0u) << 23);
          last_d = e.lit && !inv ? q + k + e.hl : ~0u;
          last_o = sum;
          sum += el[j];
          nc += (ei[j] & 0xffffu) ? 1u : 0u;
        }
      }
    }
    // output positions, and the element that covers the thread's first bytes
    const uint32_t incl = wave_incl_scan_u32(sum), excl = incl - sum;
    const uint32_t ncin = wave_incl_scan_u32(nc);
    const uint64_t hm = __ballot(mask != 0);
    const uint64_t below = hm & ((1ull << lane) - 1);
    const int from = below ? 63 - __builtin_clzll(below) : 0;
    uint32_t cd = (uint32_t)__builtin_amdgcn_ds_bpermute(4 * from, (int)last_d);
    uint32_t co = (uint32_t)__builtin_amdgcn_ds_bpermute(4 * from, (int)(excl + last_o));
    {
      const int top = hm ? 63 - __builtin_clzll(hm) : 0;
      const uint32_t td = (uint32_t)__builtin_amdgcn_readlane((int)last_d, top);
      const uint32_t to = (uint32_t)__builtin_amdgcn_readlane((int)(excl + last_o), top);
      if (lane == 63) *(lds_u32x4*)((lds_u32*)&s_x[par][wave][0]) = u32x4s{incl, ncin | (hm ? 0x80000000u : 0u), td, to};
    }
    __syncthreads();
    uint32_t run = op, wb = 0, ncopy = 0, copyb = 0;
#pragma unroll
    for (uint32_t w = 0; w < SB_WG / 64; ++w) {
      const u32x4s v = *(lds_u32x4*)((lds_u32*)&s_x[par][w][0]);
      if (w == wave) {
        wb = run;
        copyb = ncopy + ncin - nc;
        co = below ? co + run : cov_o;
        cd = below ? cd : cov_d;
      }
      ncopy += v.y & 0x7fffffffu;
      if (v.y >> 31) {
        cov_d = v.z;
        cov_o = run + v.w;
      }
      run += v.x;
    }
    if (run > blen) {  // (the same in every thread)
      bad = true;
      break;
    }
    const uint32_t opb = wb + excl;
    // literal data among the thread's bytes: byte k goes to k + dk[k]
    {
      uint32_t litm = cd <= q ? 0xffffu : (cd - q < SB_BYTES ? (0xffffu << (cd - q)) : 0u);
      uint32_t dk[SB_BYTES];
#pragma unroll
      for (uint32_t k = 0; k < SB_BYTES; ++k) dk[k] = co + q - cd;
      uint32_t o = opb, mk = mask;
#pragma unroll
      for (int j = 0; j < SB_EL; ++j) {
        if (mk) {
          mk &= mk - 1;
          const uint32_t k = (ei[j] >> 16) & 15u, a = k + ((ei[j] >> 20) & 7u);
          const bool lit = (ei[j] >> 23) & 1u;
          litm &= (1u << k) - 1u;
          if (lit) litm |= 0xffffu << a;
          const uint32_t d = o - a;
#pragma unroll
          for (uint32_t kk = 0; kk < SB_BYTES; ++kk) dk[kk] = kk >= k ? d : dk[kk];
          o += el[j];
        }
      }
      litm &= (1u << inb) - 1u;
      if (__ballot(litm != 0xffffu || mask) == 0) {
        // 16 bytes of one literal in every lane: aligned dwords, and bytes at
        // the ends
        const uint32_t D = dk[0] & (OUT - 1), r = D & 3;
        lds_u32* o32 = (lds_u32*)out + (D >> 2);
        if (__ballot(r) == 0) {
          o32[0] = w0; o32[1] = w1; o32[2] = w2; o32[3] = w3;
        } else {
          const uint32_t s = (4 - r) & 3;  // dword 1 starts at byte 4 - r (r > 0)
          if (r == 0) {
            o32[0] = w0;
          } else {
#pragma unroll
            for (uint32_t k = 0; k < 3; ++k)
              if (k + r < 4) out[D + k] = (uint8_t)(w0 >> (8 * k));
          }
          o32[1] = r ? __builtin_amdgcn_alignbyte(w1, w0, s) : w1;
          o32[2] = r ? __builtin_amdgcn_alignbyte(w2, w1, s) : w2;
          o32[3] = r ? __builtin_amdgcn_alignbyte(w3, w2, s) : w3;
#pragma unroll
          for (uint32_t k = 13; k < 16; ++k)
            if (k + r >= 16) out[D + k] = (uint8_t)(w3 >> (8 * (k - 12)));
        }
      } else {
#pragma unroll
        for (uint32_t k = 0; k < SB_BYTES; ++k) {
          const uint32_t w = k < 4 ? w0 : k < 8 ? w1 : k < 12 ? w2 : w3;
          if ((litm >> k) & 1u) out[(dk[k] + k) & (OUT - 1)] = (uint8_t)(w >> (8 * (k & 3)));
        }
      }
    }
    // copies, in the order of the output, SB_LIST at a time
    for (uint32_t base = 0; base < ncopy; base += SB_LIST) {
      {
        uint32_t o = opb, poff = 0, rs = 0, c = copyb - base;
        uint32_t po = 0, pn = 0, ps = 0;  // the thread's last copy without a period: output position, bytes, source
#pragma unroll
        for (int j = 0; j < SB_EL; ++j) {
          const uint32_t off = ei[j] & 0xffffu, n = el[j];
          if (off) {
            if (off != poff || off > 64) rs = o;  // the run of copies with this offset starts here
            const bool wrap = o + n - rs > off;   // the source would reach past the run's start
            uint32_t src_o = wrap ? rs - off : o - off;
            // bytes of the copy before: from where that one takes them
            if (!wrap && src_o - po < pn && src_o - po + n <= pn) src_o = ps + (src_o - po);
            po = o;
            ps = src_o;
            pn = wrap ? 0u : n;
            if (off > rs) bad = true;
            else if (c < SB_LIST)
              s_list[c] = u32x2s{o | (src_o << 16), n | (wrap ? (off << 8) | (((o - rs) % off) << 16) : 0u)};
            if (off > rs) {
              pn = 0;
              if (c < SB_LIST) s_list[c] = u32x2s{0u, 0u};
            }
            ++c;
          }
          poff = off;
          o += n;
        }
      }
      __syncthreads();
      const uint32_t cnt = min(ncopy - base, SB_LIST);
      uint32_t ex[2], ey[2];
      bool pend[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const uint32_t i = u * SB_WG + tid;
        const u32x2s e = i < cnt ? s_list[i] : u32x2s{0u, 0u};
        ex[u] = e.x;
        ey[u] = e.y;
        pend[u] = false;
        const uint32_t n = e.y & 0x7fu, per = (e.y >> 8) & 0x7fu, o = e.x & 0xffffu, so = e.x >> 16;
        if (n) {
          if (so + (per ? per : n) <= fin) {
            snap_copy(out, o, so, n, per, e.y >> 16);
          } else {
            pend_mark<true>(s_pend, o, n);
            pend[u] = true;
          }
        }
      }
      __syncthreads();
      while (__ballot(pend[0] || pend[1])) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const uint32_t n = ey[u] & 0x7fu, per = (ey[u] >> 8) & 0x7fu, o = ex[u] & 0xffffu, so = ex[u] >> 16;
          if (pend[u] && !pend_any(s_pend, so, per ? per : n)) {
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
            snap_copy(out, o, so, n, per, ey[u] >> 16);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
            pend_mark<false>(s_pend, o, n);
            pend[u] = false;
          }
        }
      }
      __syncthreads();
    }
    if (ncopy == 0) __syncthreads();
    // the output that became final goes to memory, 16 bytes at a time
    const bool lastp = A + SB_PASS >= qe;
    fin = run;
    if (cov_d != ~0u && !lastp) fin = min(run, cov_o + (A + SB_PASS > cov_d ? A + SB_PASS - cov_d : 0u));
    const uint32_t upto = lastp ? (run + 15u) & ~15u : fin & ~15u;
    for (uint32_t x = flushed + 16 * tid; x < upto; x += 16 * SB_WG)
      *reinterpret_cast<u32x4s*>(dst + x) = *(lds_u32x4*)((lds_u32*)&s_out[0] + (x >> 2));
    flushed = upto;
    op = run;
  }
  if (op != blen) bad = true;
  if (bad) set_err(err, ERR_SNAPPY, p);
}

template __global__ void k_snappy_blk<SNAP_SHAPE[0]>(const ColScan*, SegTable, uint8_t*, uint32_t*, int);
template __global__ void k_snappy_blk<SNAP_SHAPE[1]>(const ColScan*, SegTable, uint8_t*, uint32_t*, int);
template __global__ void k_snappy_blk<SNAP_SHAPE[2]>(const ColScan*, SegTable, uint8_t*, uint32_t*, int);

}  // namespace pqk
